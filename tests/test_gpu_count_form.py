"""At-least-t constraints in the count form (csrc/count_kernel.h) against the
oracle: lengths at the edges of every segment shape, thresholds on both sides of
the middle (where the false literals are counted instead), points inside, on
the faces and outside the box, grouped and per-bin launches, the fused check."""
import numpy as np
import pytest

import oracle
from gpu_cases import TOL32, errors, to_np
from workloads import assemble

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"
LENGTHS = (3, 4, 5, 8, 9, 12, 13, 16, 17, 24, 25, 32, 33, 47, 48, 49, 63, 64, 65, 95, 96, 97, 126, 127)


@pytest.fixture(scope="module")
def ffs():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_15020_amd as P
    P.lib()
    return P


def instance(seed=5, n=200):
    rng = np.random.default_rng(seed)
    groups = []
    for k in LENGTHS:
        for t in sorted({2, k // 4, k // 2, (k + 1) // 2, (k + 2) // 2, k // 2 + 2, k - 1}):
            if not 2 <= t <= k - 1:
                continue
            v = rng.choice(n, size=k, replace=False) + 1
            groups.append((2, [t], [np.where(rng.random(k) < 0.5, -v, v).astype(np.int32)]))
    inst = assemble(n, groups)
    inst.weights = rng.uniform(0.5, 1.5, inst.m).astype(np.float32)
    return inst


@pytest.mark.parametrize("dist", ["uniform", "settled", "face", "outside"])
@pytest.mark.parametrize("B", [1, 16, 33, 130])
def test_against_oracle(ffs, dist, B):
    inst = instance()
    rng = np.random.default_rng(B)
    x = rng.uniform(-1, 1, (inst.n_vars, B))
    if dist == "settled":
        x = np.where(rng.random(x.shape) < 0.8, np.sign(x), x)
    elif dist == "face":
        x = np.sign(x)
    elif dist == "outside":
        x = 1.1 * x
    x = np.ascontiguousarray(x.astype(np.float32))
    ref = oracle.eval_batch(inst, x.astype(np.float64), want_con=True)
    chk = oracle.check(inst, x.astype(np.float64))
    # outside the box the terms grow with the products of |l|: the oracle's own scale
    scale = max(1.0, float(np.abs(ref["con_val"]).max()))
    prob = ffs.Problem(inst)
    for mode in ("group_all", "per_bin", "group_dft"):
        plan = ffs.Plan(prob, B, mode=mode)
        assert all(b["class"] == "count" and b["fg"] == 1 for b in plan.describe()["bins"]["f32"])
        out = to_np(plan.eval(torch.from_numpy(x).to(DEV), want_con=True, want_check=True))
        e = errors(inst, out, ref)
        assert max(e.values()) <= TOL32 * scale, (mode, e)
        assert np.array_equal(out["n_sat"], chk["n_sat"]) and np.array_equal(out["U"], chk["U"])
        plan.close()
