"""FP64 evaluation of few root-of-unity constraints: frequencies split over four
waves up to 256 units in all, one wave a unit beyond; a single bin in a launch of its
own. Against the oracle on both sides of each rule."""
import numpy as np
import pytest

import oracle
from gpu_cases import TOL64, errors, to_np
from workloads import assemble

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("lens,B,split,grouped", [
    ((20,), 1, False, False), ((31,), 64, False, False), ((32,), 1, True, False), ((79,), 16, True, False),
    ((80,), 64, True, False), ((512,), 5, True, False), ((33, 79, 80, 100, 300, 512), 1, True, True),
    ((20, 100), 64, True, True), ((100,) * 32, 64, True, True), ((100,) * 33, 64, False, True),
    ((512,) * 64, 16, True, True), ((512,) * 64, 17, False, True)])
def test_few_units(lens, B, split, grouped):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_15020_amd as ffs
    rng = np.random.default_rng(len(lens) + B)
    n = 640
    groups = []
    for k in lens:
        v = rng.choice(n, size=k, replace=False) + 1
        groups.append((2, [max(2, k // 2 - 3)], [np.where(rng.random(k) < 0.5, -v, v).astype(np.int32)]))
    inst = assemble(n, groups)
    inst.weights = rng.uniform(0.5, 1.5, inst.m).astype(np.float32)
    plan = ffs.Plan(ffs.Problem(inst), B)
    bins = plan.describe()["bins"]["f64"]
    assert all(b["fg"] == (4 if split and b["maxk"] >= 32 else 1) for b in bins), bins
    assert all(b["in_group64"] == grouped for b in bins)
    x = rng.uniform(-1, 1, (n, B))
    x = np.where(rng.random((n, B)) < 0.3, np.sign(x), x)
    out = to_np(plan.eval(torch.from_numpy(x).to(DEV), want_con=True))
    ref = oracle.eval_batch(inst, x, want_con=True)
    e = errors(inst, out, ref)
    assert max(e.values()) <= TOL64, e
