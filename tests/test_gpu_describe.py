"""The pulled gradient in a plan's description: chunks of variables, and the objective
rows of four chunks each."""
import pytest

import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pull,vc,chunks", [("auto", 0, 131), ("le3", 4, 33), ("le7", 8, 17), ("off", 0, 0)])
def test_pulled_gradient_is_described(pull, vc, chunks):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_15020_amd as ffs
    inst = workloads.random_hybrid(131, 8, n_or=500, or_len=(1, 3))
    d = ffs.Plan(ffs.Problem(inst), 9, pull=pull, pull_vc=vc).describe()
    assert d["pull_chunks"] == chunks and d["pull_rows"] == -(-chunks // 4)
    if chunks:
        assert d["objective_rows"] == d["pull_rows"]
