"""The count form and the frequencies chosen at the point where they end and where
points are not numbers: constraints of exactly the longest length of the count
form and one more, NaN and infinite points (which stay with their restart), the
fused check of such points, and the rounding between batches of different
composition."""
import numpy as np
import pytest

import oracle
from gpu_cases import TOL32, TOL64, errors, to_np, var_scale
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


def instance(lengths, seed, n=600):
    rng = np.random.default_rng(seed)
    groups = []
    for k in lengths:
        for t in sorted({2, k // 4 + 1, k // 2, k // 2 + 2, k - 1}):
            if not 2 <= t <= k - 1:
                continue
            v = rng.choice(n, size=k, replace=False) + 1
            groups.append((2, [t], [np.where(rng.random(k) < 0.5, -v, v).astype(np.int32)]))
    inst = assemble(n, groups)
    inst.weights = rng.uniform(0.5, 1.5, inst.m).astype(np.float32)
    return inst


def settled(n, B, rng):
    u = rng.uniform(-1, 1, (n, B))
    return np.where(rng.random((n, B)) < 0.5, np.sign(u), u).astype(np.float32)


@pytest.mark.parametrize("mode", ["group_all", "per_bin"])
@pytest.mark.parametrize("B", [1, 40])
def test_longest_count_form(ffs, B, mode):
    inst = instance((126, 127, 128, 129, 150), 3)
    plan = ffs.Plan(ffs.Problem(inst, fp64_min_len=200), B, mode=mode)
    classes = {(b["class"], b["ct"]) for b in plan.describe()["bins"]["f32"]}
    assert classes == {("count", "f32"), ("dft", "f32")}
    assert max(b["maxk"] for b in plan.describe()["bins"]["f32"] if b["class"] == "count") == 128
    x = settled(inst.n_vars, B, np.random.default_rng(B))
    ref = oracle.eval_batch(inst, x.astype(np.float64), want_con=True)
    out = to_np(plan.eval(torch.from_numpy(x).to(DEV), want_con=True))
    assert max(errors(inst, out, ref).values()) <= TOL32


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("lengths", [(3, 4, 9, 16, 17, 32, 33, 64, 100, 127), (80, 128, 200, 257, 512)])
@pytest.mark.parametrize("dt", [torch.float32, torch.float64])
def test_bad_restart_leaves_the_others(ffs, bad, lengths, dt):
    inst = instance(lengths, 5)
    B, col = 21, 6
    good = settled(inst.n_vars, B, np.random.default_rng(2))
    x = good.copy()
    var = 17
    x[var, col] = bad
    plan = ffs.Plan(ffs.Problem(inst), B)
    out = to_np(plan.eval(torch.from_numpy(x).to(DEV, dt), want_con=True))
    keep = [b for b in range(B) if b != col]
    ref = oracle.eval_batch(inst, np.ascontiguousarray(x[:, keep]).astype(np.float64), want_con=True)
    e = errors(inst, out, ref, cols=keep)
    assert max(e.values()) <= (TOL32 if dt == torch.float32 else TOL64), e
    holds = np.array([var + 1 in np.abs(inst.lits[inst.con_ptr[c]:inst.con_ptr[c + 1]]) for c in range(inst.m)])
    assert holds.any() and not np.isfinite(out["con_val"][holds, col]).any()
    assert np.isfinite(out["con_val"][~holds, col]).all() and not np.isfinite(out["F"][col])
    if dt == torch.float32:   # the fused check rounds the point: NaN is False, -inf True
        chk = to_np(plan.eval(torch.from_numpy(x).to(DEV), want_con=True, want_check=True))
        want = oracle.check(inst, np.nan_to_num(x, nan=1.0).astype(np.float64))
        for k in ("n_sat", "U"):
            assert np.array_equal(chk[k], want[k]), k


def test_count_form_is_a_restarts_own(ffs):
    """FP32 at-least-t up to 128 literals: a restart's values and gradient are the
    same bits alone, in a batch, in another column and beside a bad restart."""
    inst = instance((3, 4, 9, 16, 17, 32, 33, 64, 100, 127), 7)
    prob = ffs.Problem(inst)
    x = settled(inst.n_vars, 37, np.random.default_rng(3))

    def run(xx):
        return to_np(ffs.Plan(prob, xx.shape[1]).eval(torch.from_numpy(np.ascontiguousarray(xx)).to(DEV), want_con=True))
    full = run(x)
    alone = run(x[:, 5:6])
    moved = run(x[:, ::-1])
    y = x.copy()
    y[:, 6] = np.nan
    beside = run(y)
    for k in ("con_val", "grad"):
        assert np.array_equal(full[k][:, 5], alone[k][:, 0]), k
        assert np.array_equal(full[k], moved[k][:, ::-1]), k
        assert np.array_equal(full[k][:, 5], beside[k][:, 5]), k


def test_chosen_frequencies_round_within_the_parity_bound(ffs):
    """Frequencies chosen at the point are those of the restarts of a wave together:
    beside other restarts a result may round differently. FP64: twice the error
    against the oracle, 2e-12 at natural scale. FP32: each slot is one rounding of
    nearly the same FP64 value, at most one unit in the last place of a value up to
    the weight, 2^-23; an objective row and its split's sum round once each."""
    inst = instance((80, 128, 200, 257, 400, 512), 9)
    prob = ffs.Problem(inst)
    x = settled(inst.n_vars, 33, np.random.default_rng(4))
    S = var_scale(inst)
    wsum = float(np.abs(inst.weights).sum())
    for dt, ulp in ((torch.float32, 2.0 ** -23), (torch.float64, 2 * TOL64)):
        def run(xx):
            xx = torch.from_numpy(np.ascontiguousarray(xx)).to(DEV, dt)
            return to_np(ffs.Plan(prob, xx.shape[1]).eval(xx, want_con=True))
        full, again = run(x), run(x)
        assert all(np.array_equal(full[k], again[k]) for k in full)   # the same batch: the same bits
        y = x.copy()
        y[:, 6] = np.nan
        z = x.copy()
        z[:, 6] *= 1.5
        for other, cols in ((run(x[:, 5:6]), [0]), (run(y), [5]), (run(z), [5]), (run(x[:, ::-1]), [27])):
            assert np.max(np.abs(other["con_val"][:, cols[0]] - full["con_val"][:, 5])) <= ulp
            assert np.all(np.abs(other["grad"][:, cols[0]] - full["grad"][:, 5]) <= 2 * ulp * S)
            assert abs(other["F"][cols[0]] - full["F"][5]) <= 4 * ulp * wsum
