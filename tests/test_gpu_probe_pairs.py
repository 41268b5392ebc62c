"""The SoA probe reads the two x corners of a pair together: particles whose
pair lies in one package, across a package face, in the far field, on and
past the domain's faces, in both precisions, against the packed probe (the
same blend from single-corner reads)."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [4, 36, 68])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_pairs_match_packed(N, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_11473_amd as sg
    from paper_2512_11473_amd import workload
    h = 1.0 / N
    rng = np.random.default_rng(N)
    i = rng.integers(-3, N + 3, (6000, 3))
    pos = (i + rng.choice([0.0, 0.5, 0.25, 0.75, 0.999], i.shape)) * h      # on data points, cell faces and between
    wl = workload.setup(synth.sphere((0.5, 0.5, 0.5), 0.45), N, 0.1, 2, dtype=dtype, particles=pos)
    sg.compute_gradient(wl.grid, wl.phi, wl.grad)
    sg.probe_particles(wl.grid, wl.phi, wl.grad, wl.pos, wl.phi_p, wl.nrm_p)
    packed = torch.empty((wl.grid.n_total, 64, 4), dtype=dtype, device="cuda")
    sg.compute_gradient_packed(wl.grid, wl.phi, packed)
    p, n = torch.empty_like(wl.phi_p), torch.empty_like(wl.nrm_p)
    sg.probe_particles_packed(wl.grid, packed, wl.pos, p, n)
    eps = torch.finfo(dtype).eps
    # eight products and sums of values up to B = 16 h on either side
    assert float((p - wl.phi_p).abs().max()) <= 32 * eps * 16 * h
    # the same for g (up to 16), then g / |g|: compared where g is not small
    big = (wl.nrm_p.norm(dim=1) > 0.5) & (n.norm(dim=1) > 0.5)
    assert torch.equal(wl.nrm_p.norm(dim=1) > 0.5, n.norm(dim=1) > 0.5)
    assert N == 4 or int(big.sum()) > 100
    near = big & (p.abs() < 4 * h)
    assert float((n - wl.nrm_p)[near].abs().max() if bool(near.any()) else 0.0) <= 32 * eps * 16 / 0.05
