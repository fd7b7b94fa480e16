"""The slot reduction at every access width (1, 2 or 4 restarts per access, by
the batch's divisor and the buffers' alignment): gradients against the oracle,
and the step against the gradient, at batches around the widths and the block."""
import numpy as np
import pytest

import oracle
from gpu_cases import TOL32, TOL64, errors, to_np
from workloads import random_hybrid

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("B", [1, 2, 3, 4, 6, 63, 64, 126, 128, 255, 256, 258, 260, 512, 514])
def test_widths(B):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_15020_amd as P
    # variables of 0 .. many occurrences: batches of 8 and their remainders
    inst = random_hybrid(37, 5, n_or=60, or_len=(1, 9), n_xor=10, xor_len=(1, 20), n_card=8, card_len=(5, 30), weights="uniform")
    rng = np.random.default_rng(B)
    x = rng.uniform(-1, 1, (inst.n_vars, B)).astype(np.float32)
    ref = oracle.eval_batch(inst, x.astype(np.float64), want_con=False)
    plan = P.Plan(P.Problem(inst), B)
    for dt, tol in ((torch.float32, TOL32), (torch.float64, TOL64)):
        out = to_np(plan.eval(torch.from_numpy(x).to(DEV, dt)))
        e = errors(inst, out, ref)
        assert max(e.values()) <= tol, (dt, e)
    # a point buffer at each 4-byte offset: the step falls back to narrower accesses
    g = plan.eval(torch.from_numpy(x).to(DEV))["grad"]
    for off in range(4):
        buf = torch.zeros(inst.n_vars * B + off, device=DEV)
        xt = buf[off:].view(inst.n_vars, B)
        xt.copy_(torch.from_numpy(x))
        plan.run_steps(xt, 1, 0.125)
        want = torch.clamp(torch.addcmul(torch.from_numpy(x).to(DEV, torch.float64), g.double(), torch.tensor(-0.125, device=DEV, dtype=torch.float64)), -1, 1)
        assert torch.max(torch.abs(xt.double() - want)).item() <= 2.0 ** -24 * 2
