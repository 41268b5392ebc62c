"""The sweeps' and the Laplacian's 64-bit byte offsets, taken by fields of more
than 4 GiB: every cell of a grid activated, so that the field just exceeds
them.  The sweeps of every configuration that chooses the offsets' width, and a
batch of the one grid, against the LDS row exchange, which always has 64-bit
offsets: the same update, so the same bits.  The Laplacian of the last package
layers against differences of the dense field."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,M", [(torch.float32, 257), (torch.float64, 204)], ids=["f32", "f64"])
def test_fields_beyond_4_gib(dtype, M):
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

    def swept(variant, n_iter):
        sg.set_sweep_config(variant, 1)
        phi = start.clone()
        sg.reinitialize(g, phi, scratch, n_iter)
        return phi

    try:
        want = swept(5, 3)
        assert not torch.equal(want, start)
        for variant in (0, 3, 7):
            assert torch.equal(swept(variant, 3), want), variant
    finally:
        sg.set_sweep_config(0, 1)
    if dtype == torch.float32:
        batch = sg.Batch([g])
        phi = start.clone()
        batch.reinitialize(phi, scratch, 3, use_graph=False)
        assert torch.equal(phi, want)
        batch.destroy()

    # up to seven roundings of sums of at most 76 h (six normal deviates and
    # six times one, each below 6.3 h); in FP64 the reference makes them too
    sg.compute_laplacian(g, start, scratch)
    bar = 7 * 76 * 2.0 ** -24 if dtype == torch.float32 else 2 * 7 * 76 * 2.0 ** -53
    layers = 3

    def dense(field):   # the last package layers, [z, y, x] in float64
        f = field[(2 + (M - layers) * M * M) * 64:].view(layers, M, M, 4, 4, 4).double()
        return f.permute(0, 3, 1, 4, 2, 5).reshape(4 * layers, 4 * M, 4 * M)

    f, out = dense(start), dense(scratch)[1:-1, 1:-1, 1:-1] * g.h * g.h
    ref = (f[1:-1, 1:-1, :-2] + f[1:-1, 1:-1, 2:] + f[1:-1, :-2, 1:-1] + f[1:-1, 2:, 1:-1] + f[:-2, 1:-1, 1:-1] +
           f[2:, 1:-1, 1:-1] - 6 * f[1:-1, 1:-1, 1:-1])
    assert float((out - ref).abs().max()) <= bar * g.h
    g.destroy()
