"""The default sweep configuration takes Morton order on large fields by
itself: its results are those of the explicit id-order kernels, bit for bit,
for the sweeps (few and many, odd and even), the Laplacian, the SoA gradient and
the factorised integrals, on fields on both sides of the rule, FP32 and FP64."""
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,dtype,large", [(400, torch.float32, False), (560, torch.float32, True),
                                           (864, torch.float32, True), (1120, torch.float32, True),
                                           (608, torch.float64, True)])
def test_default_order_same_bits(N, dtype, large):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_11473_amd as sg
    from paper_2512_11473_amd import workload
    wl = workload.setup(synth.sphere((0.5, 0.5, 0.5), 0.32), N, 0.1, 2, dtype=dtype)
    g, size = wl.grid, 4 if dtype == torch.float32 else 8
    assert (g.n_total * 64 * size >= 24 << 20) == large

    def passes():
        got = []
        for n in (1, 2, 7, 8, 9):
            wl.reset()
            sg.reinitialize(g, wl.phi, wl.scratch, n)
            got.append(wl.phi.clone())
        lap = torch.empty_like(wl.phi)
        sg.compute_laplacian(g, wl.phi, lap)
        sg.compute_gradient(g, wl.phi, wl.grad)
        got += [lap, wl.grad.clone()]
        if dtype == torch.float32:
            out = torch.empty((4, g.n_core * 64), device="cuda")
            sg.compute_near_surface_integrals_factorised(g, wl.phi, wl.scratch, out)
            got.append(out)
        return got

    try:
        sg.set_sweep_config(0, 1)
        default = passes()
        sg.set_sweep_config(0, 2)       # id order at every size
        explicit = passes()
    finally:
        sg.set_sweep_config(0, 1)
    for a, b in zip(default, explicit):
        assert torch.equal(a, b)
