"""The persistent iteration loop at sizes around its mapping: one (entry, restart)
pair per thread and several, batches that do not divide the workgroup, variables
without entries, with a full batch of terms and with more than two, entries of
three and of seven literals: one iteration against the oracle, and T iterations
in one launch against the same ones in T launches, bit for bit."""
import numpy as np
import pytest

import oracle
from gpu_cases import TOL32, to_np, var_scale
from workloads import assemble

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def instance(kmax, m, n, seed):
    rng = np.random.default_rng(seed)
    groups = []
    for c in range(m):
        k = int(rng.integers(1, kmax + 1))
        # variable 1 in every third constraint, the last variable in none
        v = rng.choice(np.arange(2, n), size=k, replace=False)
        if c % 3 == 0:
            v[0] = 1
        kind = int(rng.integers(0, 2))
        groups.append((kind, [1 if rng.random() < 0.8 else k], [np.where(rng.random(k) < 0.5, -v, v).astype(np.int32)]))
    inst = assemble(n, groups)
    inst.weights = rng.uniform(0.5, 1.5, inst.m).astype(np.float32)
    return inst


@pytest.mark.parametrize("alpha", [0.0, 0.3])
@pytest.mark.parametrize("kmax,m,n,B", [(3, 1, 5, 1), (3, 48, 20, 1), (3, 49, 20, 3), (3, 120, 40, 5), (3, 130, 30, 16),
                                        (7, 52, 25, 1), (7, 60, 30, 4), (7, 150, 60, 7), (7, 100, 12, 9)])
def test_sizes(kmax, m, n, B, alpha):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_15020_amd as P
    inst = instance(kmax, m, n, 100 * m + B)
    prob = P.Problem(inst)
    plan = P.Plan(prob, B, persistent=True)
    assert plan.describe()["persistent_steps"]
    rng = np.random.default_rng(B)
    x0 = rng.uniform(-1, 1, (n, B)).astype(np.float32)
    eta = 0.05
    x = torch.from_numpy(x0).to(DEV)
    out = to_np(plan.run_iters(x, 1, eta, alpha))
    ref = oracle.eval_batch(inst, x0.astype(np.float64))
    rc = oracle.check(inst, x0.astype(np.float64))
    wsum = float(np.abs(inst.weights).sum())
    assert np.max(np.abs(out["F"] - ref["F"])) / wsum <= TOL32
    want = np.clip(x0 - eta * ref["g"], -1, 1)
    assert np.max(np.abs(x.cpu().numpy() - want) / (eta * np.maximum(var_scale(inst)[:, None], 1.0))) <= TOL32 + 1e-5
    assert np.array_equal(out["n_sat"], rc["n_sat"]) and np.array_equal(out["U"], rc["U"])
    res = []
    for parts in ([4], [1, 1, 1, 1]):
        prob.set_weights(inst.weights)
        x = torch.from_numpy(x0).to(DEV)
        for T in parts:
            out = to_np(plan.run_iters(x, T, eta, alpha))
        res.append((x.cpu().numpy(), out, prob.get_weights().cpu().numpy()))
    (xa, oa, wa), (xb, ob, wb) = res
    assert np.array_equal(xa, xb) and np.array_equal(wa, wb)
    assert all(np.array_equal(oa[q], ob[q]) for q in ("F", "n_sat", "U"))
