"""One step in place through the pulled gradient (the stepped points come back in the
launch of the sums): the same points as a step from the plan's own gradient, with
and without the optional outputs, at batch sizes of every access width."""
import pytest

import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("B", [1, 2, 3, 4, 66, 300])
def test_step_in_place(B):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_15020_amd as ffs
    inst = workloads.random_hybrid(131, 8, n_or=500, or_len=(1, 3))
    plan = ffs.Plan(ffs.Problem(inst), B)
    assert plan.describe()["pull"] == 3
    x0 = torch.from_numpy(workloads.points(inst.n_vars, B, 4)).to(DEV)
    ref = plan.eval(x0, want_check=True)
    want = plan.step(x0.clone(), ref["grad"], 0.3)
    for outs in (True, False):
        x = x0.clone()
        got = plan.eval_step(x, 0.3, want_F=outs, want_check=outs)
        assert torch.equal(x, want)
        for k, v in got.items():
            assert torch.equal(v, ref[k]), k
    off = torch.empty(inst.n_vars * B + 1, device=DEV)[1:].view(inst.n_vars, B)   # a buffer aligned to 4 bytes only
    off.copy_(x0)
    plan.eval_step(off, 0.3)
    assert torch.equal(off, want)
