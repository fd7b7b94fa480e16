"""Gradients of the learned initialiser at the sizes its partial sums turn at: a wide
net whose partials do not fit the buffer at once (it is summed early and used again
within the pass; 64 slices of the constraints), and the deepest net (as many sums
in one launch as there can be, row counts that are no multiple of a slice).
Against the reference with bfloat16 operands. The device differs from it by
operands that round to the other neighbour, a subset of the roundings by which the
reference differs from FP64: the tolerance is that difference, and not below
the 2e-2 of tests/test_gpu_mpnn.py."""
import numpy as np
import pytest

import workloads
from oracle import mpnn_ref

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("H,R,n,m", [(256, 2, 2000, 8300), (32, 8, 150, 333), (32, 1, 1, 1)])
def test_gradients(H, R, n, m):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_15020_amd as ffs
    from paper_2308_15020_amd.mpnn import Mpnn
    inst = workloads.random_hybrid(n, 3, n_or=m, or_len=(1, 1) if n == 1 else (2, 3))
    prob = ffs.Problem(inst)
    net = Mpnn(H, R, device=0, seed=1)
    p = mpnn_ref.init_params(H, R, seed=5)
    rng = np.random.default_rng(6)
    for name, shp in mpnn_ref.param_shapes(H, R):
        if len(shp) == 1 and name != "wo":
            p[name] = rng.uniform(-0.1, 0.1, shp)
    flat = mpnn_ref.flatten(p, H, R).astype(np.float32)
    net.set_params(flat)
    p = mpnn_ref.unflatten(flat.astype(np.float64), H, R)
    g = mpnn_ref.Graph(inst)
    tgt = np.where(rng.random(n) < 0.5, -0.8, 0.8).astype(np.float32)
    loss = float(net.backward(prob, torch.from_numpy(tgt).to(DEV)).item())
    got = net.grads()
    again = (net.backward(prob, torch.from_numpy(tgt).to(DEV)), net.grads())[1]
    assert np.array_equal(got, again)
    l_bf, bf = mpnn_ref.backward(g, p, tgt.astype(np.float64), R, bf16=True)
    _, f64 = mpnn_ref.backward(g, p, tgt.astype(np.float64), R, bf16=False)
    assert abs(loss - l_bf) <= 1e-3 * l_bf
    dev = mpnn_ref.unflatten(got.astype(np.float64), H, R)
    scale = {k: max(np.abs(bf[k]).max(), 1e-30) for k in bf}
    tol = max(2e-2, max(np.abs(bf[k] - f64[k]).max() / scale[k] for k in bf))
    assert tol < 0.5
    errs = {k: float(np.abs(dev[k] - np.asarray(bf[k]).reshape(dev[k].shape)).max() / scale[k]) for k in bf}
    print(f"H {H} R {R}: tolerance {tol:.2e}, largest {max(errs.values()):.2e}")
    assert max(errs.values()) <= tol, errs
