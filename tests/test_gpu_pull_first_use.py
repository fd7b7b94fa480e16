"""A plan whose gradient is gathered by default brings the lists and the second
point buffer at its first gradient or step: not for checks and values, not under
the caller's capture (the slots serve there), and once per problem whichever
thread's plan is first."""
import threading

import numpy as np
import pytest

import workloads
from gpu_cases import var_scale

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


def _inst(n=200):
    return workloads.random_hybrid(n, 8, n_or=4 * n, or_len=(1, 3), n_xor=n // 10, xor_len=(2, 3))


def _x(inst, B, seed=1):
    return torch.from_numpy(workloads.points(inst.n_vars, B, seed)).to(DEV)


def test_checks_and_values_build_no_lists(ffs):
    inst = _inst()
    prob = ffs.Problem(inst)
    before = prob.info()["device_bytes"]
    plan = ffs.Plan(prob, 70)
    x = _x(inst, 70)
    assert plan.describe()["pull"] == 3
    plan.round_check(x)
    plan.round_check(x.double())
    plan.eval(x, want_grad=False)
    plan.eval(x, want_con=True)
    assert prob.info()["device_bytes"] == before and plan.describe()["pull_entries"] == 0
    plan.eval(x)
    assert prob.info()["device_bytes"] > before
    d = plan.describe()
    assert d["pull"] == 3 and d["pull_entries"] == inst.nnz


@pytest.mark.parametrize("call", ["eval", "eval_step", "run_steps"])
def test_first_call_under_capture_takes_the_slots(ffs, call):
    inst = _inst()
    B = 33
    prob = ffs.Problem(inst)
    plan = ffs.Plan(prob, B, use_graphs=False)
    slots = ffs.Plan(prob, B, pull="off", use_graphs=False)
    x = _x(inst, B)

    def run(p, xx):
        if call == "eval":
            return p.eval(xx)["grad"]
        if call == "eval_step":
            p.eval_step(xx, 0.1)
        else:
            p.run_steps(xx, 3, 0.1)
        return xx
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        got = run(plan, x)
    assert plan.describe()["pull_entries"] == 0
    for seed in (2, 3, 4):
        x0 = _x(inst, B, seed)
        x.copy_(x0)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, run(slots, x0.clone()))
        # eager calls of the same plan in between take the lists
        assert torch.max(torch.abs(run(plan, x0.clone()) - got)).item() <= 1e-5 * float(var_scale(inst).max())
        torch.cuda.synchronize()
    assert plan.describe()["pull_entries"] == inst.nnz


def test_plans_of_one_problem_in_several_threads(ffs):
    inst = _inst(3000)
    B = 64
    ref = ffs.Plan(ffs.Problem(inst), B).eval(_x(inst, B))["grad"].cpu()
    for _ in range(5):
        prob = ffs.Problem(inst)
        before = prob.info()["device_bytes"]
        gate = threading.Barrier(4)
        out, errs = [None] * 4, []

        def work(i):
            try:
                with torch.cuda.stream(torch.cuda.Stream()):
                    x = _x(inst, B)
                    gate.wait()
                    plan = ffs.Plan(prob, B)
                    out[i] = plan.eval(x)["grad"].cpu()
                    torch.cuda.current_stream().synchronize()
                    plan.close()
            except Exception as e:   # noqa: BLE001
                errs.append(e)
        ts = [threading.Thread(target=work, args=(i,)) for i in range(4)]
        for t in ts:
            t.start()
        for t in ts:
            t.join()
        assert not errs, errs
        assert all(torch.equal(o, ref) for o in out)
        # one set of lists: 4 words an entry, two row pointers of n + 1, 40 coefficients
        lists = 4 * (4 * inst.nnz + 2 * (inst.n_vars + 1) + 40)
        assert prob.info()["device_bytes"] - before == lists
