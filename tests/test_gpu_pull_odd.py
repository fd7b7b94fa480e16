"""Fused iterations of all-pulled plans, odd and even counts: an odd count ends
in the plan's second point buffer and the last sums' launch copies the points
back.  T iterations against T single ones, bit for bit, and against the slot
path, at batches of every access width; outputs asked for and not."""
import numpy as np
import pytest

from gpu_cases import to_np
from workloads import random_hybrid

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("use_graphs", [True, False])
@pytest.mark.parametrize("T", [1, 2, 3])
@pytest.mark.parametrize("B", [1, 6, 64, 239, 260])
def test_points_come_back(B, T, use_graphs):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_15020_amd as P
    inst = random_hybrid(53, 9, n_or=142, or_len=(1, 3))
    eta, alpha = 0.05, 0.4
    x0 = torch.from_numpy(np.random.default_rng(B).uniform(-1, 1, (53, B)).astype(np.float32)).to(DEV)
    res = {}
    for name, pull, parts in (("at once", "auto", [T]), ("singly", "auto", [1] * T), ("slots", "off", [T])):
        prob = P.Problem(inst)
        plan = P.Plan(prob, B, pull=pull, use_graphs=use_graphs)
        assert (plan.describe()["pull"] == 3) == (pull == "auto")
        x = x0.clone()
        for q in parts:
            out = plan.run_iters(x, q, eta, alpha)
        torch.cuda.synchronize()
        res[name] = (x.cpu().numpy(), to_np(out), prob.get_weights().cpu().numpy())
        plan.close()
    (xa, oa, wa), (xb, ob, wb), (xc, oc, wc) = res["at once"], res["singly"], res["slots"]
    assert np.array_equal(xa, xb) and np.array_equal(wa, wb)
    assert all(np.array_equal(oa[k], ob[k]) for k in ("F", "n_sat", "U"))
    assert np.max(np.abs(xa - xc)) <= 1e-5 and np.max(np.abs(wa - wc)) <= 1e-6
