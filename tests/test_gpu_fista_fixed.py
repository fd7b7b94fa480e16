"""FISTA at points that its step does not move (z = y): the sufficient decrease
F(z) <= F(y) holds with equality, so the first trial is accepted and eta is kept.
That takes F(y) and F(z) of one point to be the same number, also where the
weights do not add exactly: through every pull class, with few objective rows and
with more than the acceptance test adds by itself (2048)."""
import numpy as np
import pytest

import workloads

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


@pytest.mark.parametrize("pull", ["auto", "off", "le3"])
@pytest.mark.parametrize("which", ["3sat", "mixed", "many rows"])
def test_unmoved_points_keep_their_step(ffs, which, pull):
    if which == "3sat":
        inst = workloads.random_hybrid(250, 5, n_or=1050, or_len=(3, 3))
    elif which == "mixed":
        inst = workloads.config2(2000)
    else:
        inst = workloads.random_hybrid(3000, 5, n_or=30000, or_len=(3, 7))
    inst.weights = np.random.default_rng(1).uniform(0.5, 1.5, inst.m).astype(np.float32)
    B, eta = 64, 1e-3
    prob = ffs.Problem(inst)
    plan = ffs.Plan(prob, B, pull=pull)
    if which == "many rows":
        assert sum(-(-b["count"] // b["cpw"]) for b in plan.describe()["bins"]["f32"]) > 2048
    x = torch.from_numpy(np.sign(workloads.points(inst.n_vars, B, 3)).astype(np.float32)).to(DEV)
    for _ in range(400):
        plan.run_steps(x, 5, 0.5)
    g = ffs.Plan(prob, B, pull="off").eval(x)["grad"]
    still = (torch.clamp(x - eta * g, -1, 1) == x).all(0)
    assert int(still.sum()) >= B // 2
    st = plan.fista_state(x, eta)
    y = x.clone()
    plan.fista(y, st, 1)
    kept = st["eta"] == torch.tensor(eta, device=DEV)
    assert bool(kept[still].all()), int(kept[still].sum())
    assert torch.equal(y[:, still], x[:, still])
