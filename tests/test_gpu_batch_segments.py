"""A batch larger than the last-level cache is swept in segments of whole
grids: every grid bit for bit its own single-grid sweep, odd and even counts,
eager and replayed with the program's own work between the replays, with a grid
larger than a segment, many small ones and one without packages."""
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [(512, 512, 64, 512, 512, 512), (36, 1088, 48, 512), (64, 40, 128)])
def test_segments_equal_single_grids(sizes):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_11473_amd as sg
    from paper_2512_11473_amd import workload
    sg.set_sweep_config(0, 1)
    parts = [workload.setup(synth.sphere((0.5, 0.5, 0.5), 0.25 + 0.01 * k), N, 0.1, k) for k, N in enumerate(sizes)]
    empty = sg.build_packages(torch.full((8 ** 3,), 1.0, device="cuda"), 1.0 / 32)      # no packages
    fields = [p.phi0 for p in parts]
    rows = torch.empty((2, 64), device="cuda")
    sg.fill_far_field(empty, rows)
    batch = sg.Batch([parts[0].grid, empty] + [p.grid for p in parts[1:]])
    phi0 = torch.cat([fields[0], rows] + fields[1:])
    phi, scratch = phi0.clone(), torch.empty_like(phi0)
    at = [int(b) for i, b in enumerate(batch.bases) if i != 1]
    for n_iter in (4, 5):
        want = []
        for p in parts:
            p.reset()
            sg.reinitialize(p.grid, p.phi, p.scratch, n_iter)
            want.append(p.phi.clone())
        for use_graph in (False, True, True, True):
            phi.copy_(phi0)
            batch.reinitialize(phi, scratch, n_iter, use_graph=use_graph)
            torch.cuda.synchronize()
            for p, b, w in zip(parts, at, want):
                assert torch.equal(phi[b:b + p.grid.n_total], w)
            assert torch.equal(phi[int(batch.bases[1]):int(batch.bases[1]) + 2], rows)
    batch.autotune(phi0, scratch, reps=2)
    phi.copy_(phi0)
    batch.reinitialize(phi, scratch, 5)
    assert all(torch.equal(phi[b:b + p.grid.n_total], w) for p, b, w in zip(parts, at, want))
