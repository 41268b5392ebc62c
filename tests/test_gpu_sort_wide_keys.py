"""The particle sort on grids of more than 1024 coarse cells per axis, whose
Morton codes have 33 bits: the permutation is the host's stable argsort of
codes recomputed with all eleven bits of each cell coordinate."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _codes(M, pos, h):
    """Morton code of the home cell clamp(floor(x * (1/h) * 0.25), 0, M - 1), in FP32 as on the device."""
    u = pos * np.float32(1.0 / h)
    c = np.fmin(np.fmax(np.floor(u * np.float32(0.25)), np.float32(0)), np.float32(M - 1)).astype(np.int64)
    return sum(((c[:, a] >> b) & 1) << (3 * b + a) for a in range(3) for b in range(11))


@pytest.mark.parametrize("M", [1024, 1025, 1625])
def test_sort_wide_keys(M):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_11473_amd as sg
    h = 0.25 / M
    grid = sg.build_packages(torch.full((M ** 3,), 1.0, device="cuda"), h)
    rng = np.random.default_rng(M)
    for n in (1, 4097, 50021):
        pos = rng.random((n, 3)).astype(np.float32)
        pos[: n // 3] = (1.0 - 3.0 * h * rng.random((n // 3, 3))).astype(np.float32)   # the last cells, many equal keys
        pos[n // 3: n // 2, 0] = (1.0 - 40.0 * h * rng.random(n // 2 - n // 3)).astype(np.float32)
        pt = torch.from_numpy(pos).cuda()
        ps, perm = torch.empty_like(pt), torch.empty(n, dtype=torch.int32, device="cuda")
        sg.sort_particles(grid, pt, ps, perm)
        want = np.argsort(_codes(M, pos, h), kind="stable")
        assert np.array_equal(perm.cpu().numpy().view(np.uint32).astype(np.int64), want)
        assert np.array_equal(ps.cpu().numpy().view(np.uint32), pos[want].view(np.uint32))
    grid.destroy()
