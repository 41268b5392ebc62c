"""The 64-bit byte offsets of the sweeps with several sets per wavefront, in id
order and in Morton order, on fields of more than 4 GiB (every cell of a grid
activated): the bits of the LDS row exchange, which always has 64-bit offsets.
Id order on fields this large is (0, 2) and more; (0, 1) takes Morton order."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,M", [(torch.float32, 257), (torch.float64, 204)], ids=["f32", "f64"])
def test_groups_beyond_4_gib(dtype, M):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2512_11473_amd as sg
    g = sg.build_packages(torch.zeros(M ** 3, device="cuda"), 1.0 / (4 * M))
    size = torch.empty(0, dtype=dtype).element_size()
    assert g.n_packages == M ** 3 and g.n_total * 64 * size > 1 << 32
    gen = torch.Generator(device="cuda").manual_seed(M)
    start = torch.randn(g.n_total * 64, device="cuda", dtype=dtype, generator=gen) * g.h
    sg.fill_far_field(g, start)
    scratch = torch.empty_like(start)

    def swept(variant, groups):
        sg.set_sweep_config(variant, groups)
        phi = start.clone()
        sg.reinitialize(g, phi, scratch, 2)
        return phi

    try:
        want = swept(5, 1)
        assert not torch.equal(want, start)
        for variant, groups in ((0, 2), (0, 3), (0, 4), (0, 8), (3, 2), (3, 8)):
            assert torch.equal(swept(variant, groups), want), (variant, groups)
    finally:
        sg.set_sweep_config(0, 1)
    g.destroy()
