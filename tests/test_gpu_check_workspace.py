"""The exact check alone works in the memory that a plan holds from its creation,
for points of either type: nothing is allocated for it, so that a first call may be
captured, and evaluations before and after it are unchanged."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_cases import to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n,m,B", [(400, 3, 1), (400, 3, 2), (97, 300, 64), (97, 300, 65), (300, 40, 300)])
def test_no_memory_of_its_own(n, m, B):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_15020_amd as ffs
    inst = workloads.random_hybrid(n, 3, n_or=m, or_len=(2, 6))
    plan = ffs.Plan(ffs.Problem(inst), B)
    rows, splits = m + n, -(-(m + n) // 64)
    stride = -(-B // 64)
    signs = 8 * n * (1 if stride == 1 else -(-stride // 4) * 4)
    # slots, objective rows and their sums, count rows and their sums
    held = 4 * B * inst.nnz + max(4 * B * rows, signs) + 4 * B * splits + 4 * B * rows + 4 * B * splits
    assert plan.describe()["device_bytes"] == held
    xn = workloads.points(n, B, 5)
    x = torch.from_numpy(xn).to(DEV)
    xd = x.double()
    before = to_np(plan.eval(x, want_con=True))
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        cap = plan.round_check(xd)
    for _ in range(3):
        for t in cap.values():
            t.zero_()
        g.replay()
        torch.cuda.synchronize()
        eager = to_np(plan.round_check(x))
        ref = oracle.check(inst, xn.astype(np.float64))
        for name in ("n_sat", "U"):
            assert np.array_equal(eager[name], ref[name])
        for name, v in to_np(cap).items():
            assert np.array_equal(v, eager[name]), name
        after = to_np(plan.eval(x, want_con=True))
        assert all(np.array_equal(after[k], before[k]) for k in before)
    assert plan.describe()["device_bytes"] == held
