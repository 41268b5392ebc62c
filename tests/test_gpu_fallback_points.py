"""The plain fallback of the learned integrals at few and odd numbers of listed
points: the upper bound of the accepted range is put between two of the
network's own values, so that a chosen number of points falls back, and these
must carry the plain kernel's bits, the others the network's."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def case():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2512_11473_amd as sg
    from test_gpu_mlp import _sphere_grid, init_params
    wl = _sphere_grid(sg)[1]
    n = wl.grid.n_core * 64
    plain = torch.empty((4, n), device="cuda")
    sg.compute_near_surface_integrals(wl.grid, wl.phi, plain)
    unsat = torch.empty(n, dtype=torch.uint8, device="cuda")
    x = torch.empty((n, 216), device="cuda")
    sg.gather_windows(wl.grid, wl.phi, x, unsat)
    model = sg.Mlp(init_params(11))
    y = torch.empty((n, 4), device="cuda")
    model.forward(x, y)
    return sg, wl, model, plain, unsat.bool(), y.t().contiguous()


@pytest.mark.parametrize("k", [0, 1, 2, 15, 16, 17, 33, 64, 1000])
def test_listed_points_carry_the_plain_value(case, k):
    sg, wl, model, plain, unsat, y = case
    kw = y[0][unsat].sort(descending=True).values
    model.set_gate(3.0e38, -1e30, float(kw[k]))
    out = torch.empty_like(plain)
    nf = torch.zeros(1, dtype=torch.int32, device="cuda")
    sg.compute_near_surface_integrals(wl.grid, wl.phi, out, model=model, n_fallback=nf)
    listed = unsat & (y[0] > kw[k])
    assert int(nf.item()) == int(listed.sum().item()) <= k
    assert torch.equal(out[:, listed], plain[:, listed])
    net = unsat & ~listed
    assert torch.equal(out[:, net], y[:, net])
    assert torch.equal(out[:, ~unsat], plain[:, ~unsat])
