"""The pulled gradient with a weight that is not finite: it reaches the variables
of its own constraint, as through the slots, and no others (the lists' null
entries read the weight of constraint 0)."""
import numpy as np
import pytest

import workloads
from gpu_cases import var_scale

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def ffs():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_15020_amd as P
    P.lib()
    return P


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("pull,lens", [("auto", (3, 3)), ("le7", (2, 7))])
@pytest.mark.parametrize("B", [5, 300])
def test_one_weight_stays_with_its_constraint(ffs, bad, pull, lens, B):
    inst = workloads.random_hybrid(60, 9, n_or=150, or_len=lens)
    prob = ffs.Problem(inst)
    w = torch.ones(inst.m, device=DEV)
    w[0] = bad
    prob.set_weights(w)
    x = torch.from_numpy(workloads.points(inst.n_vars, B, 2)).to(DEV)
    plan = ffs.Plan(prob, B, pull=pull)
    assert plan.describe()["pull"] > 0
    got = plan.eval(x)["grad"].cpu().numpy()
    want = ffs.Plan(prob, B, pull="off").eval(x)["grad"].cpu().numpy()
    own = np.abs(inst.lits[inst.con_ptr[0]:inst.con_ptr[1]]) - 1
    others = np.setdiff1d(np.arange(inst.n_vars), own)
    assert np.isfinite(want[others]).all() and not np.isfinite(want[own]).any()
    # the products of the two paths round in another order (as tests/test_gpu_pull.py)
    assert np.all(np.abs(got[others] - want[others]) <= 1e-6 * var_scale(inst)[others, None])
    assert not np.isfinite(got[own]).any()
