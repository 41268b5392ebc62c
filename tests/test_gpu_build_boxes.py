"""The build's activation masks of 4 x 4 x 4 boxes of cells: the worklist is in
Morton order on grids that fill their enclosing power of two and on grids just
past one (whose last boxes are cut), and the masks take no more memory than the
grid has cells."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_11473_amd as sg
    sg.load()
    return sg


@pytest.mark.parametrize("M", [1, 2, 3, 4, 5, 8, 9, 16, 17, 33, 66, 130])
def test_worklist_order(sg, M):
    rng = np.random.default_rng(M)
    d = np.where(rng.random(M ** 3) < (0.5 if M < 10 else 0.004), 0.0, 100.0).astype(np.float32)
    d[-1] = 0.0                                        # the last cell of the last box
    g = sg.build_packages(torch.from_numpy(d).cuda(), 0.25 / M)
    t = {k: v.cpu().numpy().view(np.uint32).astype(np.int64) for k, v in g.tables().items() if v.dtype == torch.int32}
    cells = t["pkg_cell"][2:]
    c = np.stack([cells % M, (cells // M) % M, cells // (M * M)])
    code = sum(((c[a] >> b) & 1) << (3 * b + a) for a in range(3) for b in range(8))
    assert np.array_equal(t["sweep_order"], 2 + np.argsort(code, kind="stable"))
    g.destroy()


def test_memory_of_a_grid_past_a_power_of_two(sg):
    M = 513
    d = torch.full((M ** 3,), 1.0, device="cuda")
    sg.build_packages(torch.zeros(1, device="cuda"), 0.25).destroy()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    g = sg.build_packages(d, 0.25 / M)
    taken = before - torch.cuda.mem_get_info()[0]
    rows, W = M * M, (M + 63) // 64
    tables = 4 * M ** 3 + 16 * rows * ((M + 31) // 32)          # cell map, rank map
    workspace = 3 * 8 * rows * W + 8 * ((M + 3) // 4) ** 3      # bitmaps, masks
    assert taken <= 1.03 * (tables + workspace) + (16 << 20), (taken, tables, workspace)
    g.destroy()
