"""A tuned per-bin shape that splits an FP64 bin's frequencies over two waves does
not keep the bin out of the grouped launch: the tuned file does not name the
launch structure a shape was timed for, so a grouped plan may read such an entry."""
import json

import pytest

import oracle
import workloads
from gpu_cases import TOL32, errors, to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("mode", ["group_all", "group_dft", "auto"])
def test_grouped_plan_reads_a_two_way_split(tmp_path, mode):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_15020_amd as ffs
    inst = workloads.random_hybrid(600, 6, n_or=100, or_len=(3, 6), n_card=24, card_len=(130, 500))
    B = 40
    prob = ffs.Problem(inst)
    path = str(tmp_path / "tune.json")
    ffs.Plan(prob, B, mode="per_bin", autotune=True, tune_cache=path).close()
    with open(path) as f:
        cache = json.load(f)
    long_bins = [k for k in cache if "|io0|" in k and "|c1|t1|" in k]
    assert long_bins
    for k in long_bins:
        cache[k] = [1, 2, 2]
    # the automatic plan's structure as tuned: the grouped launch of every bin (2),
    # no pulled gradient, 8 constraints of a chain per wave and one wave a unit
    cache = {k: v for k, v in cache.items() if "|mode|" not in k}
    n_bins = len(ffs.Plan(prob, B).describe()["bins"]["f32"])
    cache[f"gfx950|mode|B{B}|n{inst.n_vars}|m{inst.m}|nnz{inst.nnz}|bins{n_bins}|a2|pull"] = [2, 0, 65]
    with open(path, "w") as f:
        json.dump(cache, f)
    plan = ffs.Plan(prob, B, mode=mode, autotune=True, tune_cache=path)
    d = plan.describe()
    if mode == "auto":
        assert d["tuned_modes"] == [] and d["mode"] == "group_all"   # read from the file
    fp64 = [b for b in d["bins"]["f32"] if b["class"] == "dft" and b["ct"] == "f64"]
    assert fp64 and all(b["in_group64"] and b["fg"] in (1, 4) for b in fp64)
    assert d["group64_blocks"] > 0
    x = workloads.points(inst.n_vars, B, 2)
    out = to_np(plan.eval(torch.from_numpy(x).to(DEV), want_con=True))
    ref = oracle.eval_batch(inst, x.astype("float64"), want_con=True)
    assert max(errors(inst, out, ref).values()) <= TOL32
