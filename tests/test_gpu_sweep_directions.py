"""Sweeps that alternate in direction and keep their last rows in the cache:
bands whose two buffers just exceed it (every cell of a grid activated), with
whole and ragged last workgroups, even and odd numbers of sweeps.  Against the
LDS row exchange, which always goes forward: the same update, so the same bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,M", [(torch.float32, 81), (torch.float32, 82), (torch.float64, 64),
                                     (torch.float64, 65)], ids=["f32-81", "f32-82", "f64-64", "f64-65"])
def test_alternating_sweeps(dtype, M):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2512_11473_amd as sg
    g = sg.build_packages(torch.zeros(M ** 3, device="cuda"), 1.0 / (4 * M))
    size = torch.empty(0, dtype=dtype).element_size()
    assert 1 << 28 < 2 * g.n_total * 64 * size < 1.1 * (1 << 28)
    gen = torch.Generator(device="cuda").manual_seed(M)
    start = torch.randn(g.n_total * 64, device="cuda", dtype=dtype, generator=gen) * g.h
    sg.fill_far_field(g, start)
    scratch = torch.empty_like(start)

    def swept(variant, groups, n_iter):
        sg.set_sweep_config(variant, groups)
        phi = start.clone()
        sg.reinitialize(g, phi, scratch, n_iter)
        return phi

    try:
        for n_iter in (1, 2, 9):
            want = swept(5, 1, n_iter)
            for variant, groups in ((0, 1), (0, 3), (3, 1), (3, 8), (7, 1)):
                assert torch.equal(swept(variant, groups, n_iter), want), (variant, groups, n_iter)
    finally:
        sg.set_sweep_config(0, 1)
    g.destroy()
