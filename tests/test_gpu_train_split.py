"""Training batches at the edges of the kernels' split: sixteen-sample tiles,
chunks of 64 samples, and (above 16384 samples) longer chunks with a shorter
last one.  The gradient against the FP64 oracle within the propagated
rounding error (tests/mlp_bounds.py), the output biases and the loss within
FP32 summation error, and a train step bit for bit equal to its parts."""
import numpy as np
import pytest

import mlp_bounds as mb
import oracle
from test_gpu_mlp import init_params, quantised

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_11473_amd as sg
    sg.load()
    return sg


@pytest.mark.parametrize("B", [15, 16, 17, 63, 65, 129, 4096, 4097, 4161, 16385])
def test_gradient_at_split_edges(sg, B):
    w = init_params(40)
    model = sg.Mlp(w)
    rng = np.random.default_rng(B)
    x = (rng.standard_normal((B, 216)) * 2.0).astype(np.float32)
    dy = rng.standard_normal((B, 4)).astype(np.float32)
    g = torch.empty(sg.MLP_N_PARAMS, device="cuda")
    model.backward(torch.from_numpy(x).cuda(), torch.from_numpy(dy).cuda(), g)
    q = quantised(w)
    ref = oracle.mlp_backward(q, x.astype(np.float64), dy.astype(np.float64))
    sd = mb.backward_scales(q, w.astype(np.float64), x.astype(np.float64), dy.astype(np.float64))
    got = g.double().cpu().numpy()
    z = np.abs(got - ref) / sd
    assert z.max() <= mb.K_SIGMA, (int(np.argmax(z)), z.max())
    # the output biases are FP32 sums of dy
    assert np.all(np.abs(got[-4:] - dy.astype(np.float64).sum(0)) <= 2.0 ** -23 * np.abs(dy).sum(0, dtype=np.float64))


@pytest.mark.parametrize("B", [1, 70, 4161, 16449])
def test_train_step_equals_its_parts(sg, B):
    rng = np.random.default_rng(B + 1)
    x = torch.from_numpy((rng.standard_normal((B, 216)) * 2.0).astype(np.float32)).cuda()
    t = torch.from_numpy(rng.standard_normal((B, 4)).astype(np.float32)).cuda()
    lw = np.array([1.5, 0.25, 2.0, 3.0], np.float32)
    a, b = sg.Mlp(init_params(41)), sg.Mlp(init_params(41))
    loss, y = torch.zeros(1, device="cuda"), torch.empty((B, 4), device="cuda")
    a.train_step(x, t, lw, 1e-3, loss)
    b.forward(x, y)
    e = y - t
    wo = torch.from_numpy(lw).cuda()
    g = torch.empty(sg.MLP_N_PARAMS, device="cuda")
    # (a device tensor: by a host number torch multiplies with the reciprocal)
    b.backward(x, (2.0 * wo * e) / torch.full((1,), float(B), device="cuda"), g)
    b.apply_gradient(g, 1e-3)
    for p, r in zip(a.state(), b.state()):
        assert np.array_equal(p, r)
    want = float((wo.double() * e.double() ** 2).sum())
    assert abs(float(loss) - want) <= 1e-6 * want     # a sum of positive terms, each within 4 ulp
