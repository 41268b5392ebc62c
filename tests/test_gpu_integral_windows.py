"""The plain integral kernel takes one, two or four packages per wavefront by
their number, and a window wholly on one side of the surface skips its taps:
the direct kernel, the factorised form and the field agree bit for bit on
core points at numbers of packages around those rules, and one-sided inner
packages hold the far field's constants."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,r", [(12, 0.3), (64, 0.3), (156, 0.32), (256, 0.3), (364, 0.34)])
def test_packages_per_wavefront(N, r):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_11473_amd as sg
    from paper_2512_11473_amd import workload
    wl = workload.setup(synth.sphere((0.5, 0.5, 0.5), r), N, 0.1, 5)
    g = wl.grid
    out, fact = torch.empty((4, g.n_core * 64), device="cuda"), torch.empty((4, g.n_core * 64), device="cuda")
    field, vfrac = torch.empty((g.n_total, 64, 4), device="cuda"), torch.empty_like(wl.phi)
    sg.compute_near_surface_integrals(g, wl.phi, out)
    sg.compute_near_surface_integrals_factorised(g, wl.phi, vfrac, fact)
    sg.compute_integral_field(g, wl.phi, field)
    assert torch.equal(out, fact)
    core = g.tables()["core_list"].long()
    l = torch.arange(64, device="cuda")
    i, j, k = l % 4, (l // 4) % 4, l // 16
    blocked = 8 * ((i >> 1) + 2 * (j >> 1) + 4 * (k >> 1)) + (i & 1) + 2 * (j & 1) + 4 * (k & 1)
    got = field[core][:, blocked]                                   # [n_core, 64, 4] in local order
    assert torch.equal(got.reshape(-1, 4).t(), out)
    # points whose whole support is on one side (|phi| beyond the support and the cell) hold the constants
    far = wl.phi.abs() > 6.0 * wl.h * 1.2
    far[:2] = False
    vals = torch.empty_like(field)
    vals[:, torch.arange(64, device="cuda")] = field[:, blocked]
    inside, outside = vals[far & (wl.phi < 0)], vals[far & (wl.phi > 0)]
    c_full = field[1, 0, 0]
    assert float(inside.abs().max()) == 0.0 if inside.numel() else True
    if outside.numel():
        assert torch.all(outside[:, 0] == c_full) or float((outside[:, 0] - c_full).abs().max()) <= 2.0 ** -23
        assert float(outside[:, 1:].abs().max()) == 0.0
