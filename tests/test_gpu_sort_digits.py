"""The particle sort at every digit width and pass count its plan can take
(one to four passes of 7, 8 or 9 bits, ending in the outputs or by way of
them), ragged last tiles, clustered keys and particles outside the domain:
the permutation is the host's stable argsort of the recomputed keys."""
import numpy as np
import pytest

from sort_check import assert_sorted

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_11473_amd as sg
    sg.load()
    return sg


@pytest.mark.parametrize("M", [1, 2, 5, 8, 9, 16, 33, 64, 65, 130, 256, 300, 520])
def test_sort_digit_widths(sg, M):
    h = 0.25 / M
    grid = sg.build_packages(torch.full((M ** 3,), 1.0, device="cuda"), h)
    rng = np.random.default_rng(M)
    for n in (1, 63, 4096, 8193, 50021):
        pos = rng.random((n, 3)).astype(np.float32)
        pos[: n // 3] = (0.4 + 3.0 * h * rng.random((n // 3, 3))).astype(np.float32)   # many equal keys
        pos[n // 2: n // 2 + n // 50] += np.float32(2.0) * np.sign(rng.standard_normal((n // 50, 3))).astype(np.float32)
        if n > 100:
            pos[7] = [np.nan, 0.5, np.inf]
            pos[8] = [-0.0, -np.inf, 1.0]
        pt = torch.from_numpy(pos).cuda()
        ps, perm = torch.empty_like(pt), torch.empty(n, dtype=torch.int32, device="cuda")
        need = sg.sort_workspace_bytes(grid, n)
        ws = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")[:need]
        for _ in range(2):   # the second time over the first one's workspace and outputs
            sg.sort_particles(grid, pt, ps, perm, workspace=ws if need else None)
            torch.cuda.synchronize()
            assert_sorted(M, h, pos, ps.cpu().numpy(), perm.cpu().numpy().view(np.uint32))
        assert np.array_equal(pt.cpu().numpy().view(np.uint32), pos.view(np.uint32))     # the input is only read
