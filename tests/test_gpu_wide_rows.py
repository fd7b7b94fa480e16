"""Rows of points past 2^24 bytes, and points past 2^32: the evaluation kernels
form a point's address in 64 bits there instead of one 24-bit multiply-add.
Constraints over several lanes of each kernel family (FP32 count, FP64
polynomial, chains), the last literals of the array among them; sampled
restarts against the oracle."""
import numpy as np
import pytest

import oracle
from gpu_cases import TOL32, TOL64, errors
from workloads import assemble

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dt,n,B", [("float32", 100, (1 << 22) - 64), ("float32", 100, 1 << 22), ("float32", 300, (1 << 22) + 3),
                                    ("float64", 140, (1 << 21) - 1), ("float64", 140, (1 << 21) + 5)])
def test_against_oracle(dt, n, B):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_15020_amd as P
    rng = np.random.default_rng(n)
    groups = []
    for kind, k, t in [(2, 40, 11), (0, 60, 0), (1, 45, 1), (2, 24, 12), (2, 7, 3)] + ([(2, 135, 61)] if n > 135 else []):
        v = rng.choice(n, size=k, replace=False) + 1
        groups.append((kind, [t], [np.where(rng.random(k) < 0.5, -v, v).astype(np.int32)]))
    inst = assemble(n, groups)
    torch.manual_seed(n)
    x = torch.rand(n, B, device=DEV, dtype=getattr(torch, dt)).mul_(2).sub_(1)
    cols = [0, 1, 63, 64, B // 2, B - 65, B - 2, B - 1]
    plan = P.Plan(P.Problem(inst), B)
    out = plan.eval(x, want_con=True)
    out = {q: v[..., cols].double().cpu().numpy() for q, v in out.items() if v is not None and q in ("F", "grad", "con_val")}
    ref = oracle.eval_batch(inst, x[:, cols].double().cpu().numpy(), want_con=True)
    e = errors(inst, out, ref)
    assert set(e) == {"F", "grad", "con_val"} and max(e.values()) <= (TOL32 if dt == "float32" else TOL64), e
    plan.close()
