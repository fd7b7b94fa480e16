"""The exact check alone (csrc/check.hip) against the oracle, bit for bit: word
and batch edges, constraint counts at the edges of the 64-constraint groups,
lengths on both sides of the thread / wave split, every kind, thresholds
outside [1, k], signed zeros and NaN, both point types."""
import numpy as np
import pytest

import oracle
from gpu_cases import to_np
from workloads import assemble

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"
LENGTHS = (1, 2, 3, 4, 5, 8, 31, 32, 33, 63, 64, 65, 128, 255, 256, 257, 511, 512)


@pytest.fixture(scope="module")
def ffs():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_15020_amd as P
    P.lib()
    return P


def instance(m, n, seed):
    rng = np.random.default_rng(seed)
    groups = []
    for c in range(m):
        k = min(n, LENGTHS[rng.integers(len(LENGTHS))] if c % 3 == 0 else int(rng.integers(1, 8)))
        kind = int(rng.integers(0, 3))
        prm = int(rng.integers(0, 2)) if kind == 1 else int(rng.integers(-1, k + 3))
        v = rng.choice(n, size=k, replace=False) + 1
        groups.append((kind, [prm], [np.where(rng.random(k) < 0.5, -v, v).astype(np.int32)]))
    return assemble(n, groups)


@pytest.mark.parametrize("m,n,B", [(1, 1, 1), (3, 40, 5), (31, 600, 63), (32, 600, 64), (33, 31, 65), (64, 32, 128),
                                   (65, 33, 130), (127, 600, 256), (257, 600, 257), (1000, 520, 300)])
@pytest.mark.parametrize("dt", [torch.float32, torch.float64])
def test_check_alone(ffs, m, n, B, dt):
    inst = instance(m, n, 7 * m + B)
    rng = np.random.default_rng(B)
    x = rng.uniform(-1, 1, (n, B))
    x[rng.random((n, B)) < 0.3] = -1.0
    x[0, ::2] = -0.0
    x[0, 1::3] = np.nan
    x = x.astype(np.float32)
    prob = ffs.Problem(inst)
    plan = ffs.Plan(prob, B)
    ref = oracle.check(inst, np.nan_to_num(x, nan=1.0).astype(np.float64))
    neg = x < 0
    for _ in range(2):
        out = to_np(plan.round_check(torch.from_numpy(x).to(DEV, dt)))
        assert np.array_equal(out["n_sat"], ref["n_sat"])
        assert np.array_equal(out["U"], ref["U"])
        bits = np.unpackbits(out["assign_bits"].view(np.uint8), axis=1, bitorder="little")
        assert np.array_equal(bits[:, :n].astype(bool), neg.T) and not bits[:, n:].any()
        uns = np.unpackbits(out["unsat_bits"].view(np.uint8), axis=1, bitorder="little")
        assert not uns[:, m:].any()
        assert np.array_equal(uns[:, :m].sum(0), ref["U"]) and np.array_equal(m - uns[:, :m].sum(1), ref["n_sat"])
    # each output alone
    xt = torch.from_numpy(x).to(DEV, dt)
    for name in ("assign_bits", "n_sat", "unsat_bits", "U"):
        alone = to_np(plan.round_check(xt, want=(name,)))
        assert np.array_equal(alone[name], out[name]), name
    if dt == torch.float32:   # the check beside an evaluation gives the same
        fused = to_np(plan.eval(xt, want_check=True))
        for name in ("n_sat", "unsat_bits", "U"):
            assert np.array_equal(fused[name], out[name]), name
