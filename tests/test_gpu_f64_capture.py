"""An FP64 evaluation captured by the caller and replayed after the plan was
tuned: the tuner replaces the FP32 evaluation's launch tables, the FP64
evaluation's table stays."""
import pytest

import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("B", [3, 70])
def test_captured_f64_evaluation_survives_tuning(B):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_15020_amd as ffs
    inst = workloads.random_hybrid(300, 4, n_or=200, or_len=(2, 5), n_xor=20, xor_len=(2, 9), n_card=40, card_len=(5, 200))
    plan = ffs.Plan(ffs.Problem(inst), B)
    assert any(b["in_group64"] for b in plan.describe()["bins"]["f64"])
    x = torch.from_numpy(workloads.points(inst.n_vars, B, 1)).to(DEV, torch.float64)
    out = plan.eval(x)   # the workspace, before the capture
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plan.eval(x, out=out)
    plan.tune()
    for seed in (2, 3, 4):
        x.copy_(torch.from_numpy(workloads.points(inst.n_vars, B, seed)).to(DEV, torch.float64))
        want = plan.eval(x)
        torch.cuda.synchronize()
        out["F"].zero_(), out["grad"].zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out["F"], want["F"]) and torch.equal(out["grad"], want["grad"])
