"""At-least-t constraints whose frequencies are chosen at the point
(csrc/eval_kernel.h, node_window) against the oracle: lengths at the edges of
the point counts and segment shapes, thresholds inside, at the edges of and
outside the window, points at a face, spread over a wave's restarts and outside
the box, split frequencies and per-bin launches.  Tolerances: those of the
parity tests (1e-5 and 1e-12 at natural scale)."""
import numpy as np
import pytest

import oracle
from gpu_cases import TOL32, TOL64, errors, to_np
from workloads import assemble

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


def instance(seed=3, n=640):
    rng = np.random.default_rng(seed)
    groups = []
    for k in (79, 80, 81, 96, 97, 127, 128, 129, 144, 145, 192, 193, 256, 257, 288, 289, 416, 449, 511, 512):
        for t in sorted({1, 2, k // 8, k // 4, k // 2 - 30, k // 2, k // 2 + 30, 3 * k // 4, k - 1}):
            if not 1 <= t <= k:
                continue
            v = rng.choice(n, size=k, replace=False) + 1
            sg = -1 if rng.random() < 0.5 else 1
            groups.append((2, [t], [(v * sg).astype(np.int32)]))
    inst = assemble(n, groups)
    inst.weights = rng.uniform(0.5, 1.5, inst.m).astype(np.float32)
    return inst


def pts(n, B, dist, rng):
    u = rng.uniform(-1, 1, (n, B))
    if dist == "settled":
        u = np.where(rng.random((n, B)) < 0.8, np.sign(u), u)
    elif dist == "spread":    # counts far apart within a wave
        u = np.clip(0.2 * u + np.linspace(-0.95, 0.95, B), -1, 1)
    elif dist == "face":
        u = np.sign(u) * np.where(rng.random((n, B)) < 0.02, 0.5, 1.0)
    elif dist == "outside":
        u = 1.05 * u
    return u


@pytest.mark.parametrize("dist", ["uniform", "settled", "spread", "face", "outside"])
@pytest.mark.parametrize("B", [1, 21])
def test_against_oracle(ffs, dist, B):
    inst = instance()
    x = np.ascontiguousarray(pts(inst.n_vars, B, dist, np.random.default_rng(B)).astype(np.float32))
    ref = oracle.eval_batch(inst, x.astype(np.float64), want_con=True)
    prob = ffs.Problem(inst)
    # values beyond the box grow with the product of |l|: the oracle's own scale
    scale = 1.0 if dist != "outside" else max(1.0, float(np.abs(ref["con_val"]).max()))
    for mode in ("group_all", "per_bin"):
        plan = ffs.Plan(prob, B, mode=mode)
        for dt, tol in ((torch.float32, TOL32), (torch.float64, TOL64)):
            out = to_np(plan.eval(torch.from_numpy(x).to(DEV, dt), want_con=True))
            e = errors(inst, out, ref)
            assert max(e.values()) <= tol * scale, (mode, dt, e)
        plan.close()


def test_one_nan_restart_leaves_the_others(ffs):
    inst = instance(seed=4)
    x = pts(inst.n_vars, 9, "settled", np.random.default_rng(1)).astype(np.float32)
    x[:, 4] = np.nan
    plan = ffs.Plan(ffs.Problem(inst), 9)
    out = to_np(plan.eval(torch.from_numpy(x).to(DEV), want_con=True))
    keep = [b for b in range(9) if b != 4]
    ref = oracle.eval_batch(inst, np.ascontiguousarray(x[:, keep]).astype(np.float64), want_con=True)
    e = errors(inst, out, ref, cols=keep)
    assert max(e.values()) <= TOL32, e
    assert np.isnan(out["F"][4]) and np.isnan(out["con_val"][:, 4]).all()
