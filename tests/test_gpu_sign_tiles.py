"""The sign correction's tiles on the GPU against the oracle, bit for bit, with
the round count: grid widths around the edges of a word and of a tile, signs
that travel through many tiles and launches, and values whose sign bit is not
their sign (zeros of both signs)."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sg():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2512_11473_amd as sg
    sg.load()
    return sg


@pytest.mark.parametrize("M,cores", [(1, 1), (2, 1), (17, 3), (31, 2), (32, 5), (33, 4), (63, 6), (64, 2), (65, 9),
                                     (80, 40), (97, 3), (130, 1)])
def test_tiles_match_oracle(sg, M, cores):
    rng = np.random.default_rng(M)
    d = rng.choice(np.array([3.0, -3.0, 0.5 + 1.0 / M], np.float32), M ** 3)
    at = rng.choice(M ** 3, cores, replace=False)
    d[at] = rng.choice(np.array([0.25 / M, -0.25 / M, 0.0, -0.0], np.float32), cores)
    if M > 16:   # a wall without a gap: cells behind it that no diffusion reaches keep their value
        g = d.reshape(M, M, M)
        g[:, M // 2, M // 3] = np.float32(-0.25 / M)
    ref, ref_rounds = oracle.correct_signs(M, d)
    x = torch.from_numpy(d).cuda()
    out = torch.empty_like(x)
    assert sg.correct_signs(x, 0.25 / M, out) == ref_rounds
    assert np.array_equal(out.cpu().numpy().view(np.uint32), ref.view(np.uint32))


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_points_with_signed_zeros(sg, dtype):
    from paper_2512_11473_amd import workload
    N = 68
    npd = np.float32 if dtype == torch.float32 else np.float64
    wl = workload.setup(synth.sphere((0.5, 0.5, 0.5), 0.3), N, 0.0, 0, dtype=dtype)
    run = oracle.setup(synth.sphere((0.5, 0.5, 0.5), 0.3), N, 0.0, 0, phi0_dtype=npd)
    dense = oracle.dense_state(run.tab, run.active, run.phi0, run.B)
    inner = oracle.active_points(run.tab, pkg_types=(2,))
    rng = np.random.default_rng(4)
    pick = rng.choice(inner, inner.size // 3, replace=False)
    dense[pick] = rng.choice(np.array([0.0, -0.0, 1.0, -1.0]), pick.size) * np.abs(dense[pick])
    ref, ref_rounds = oracle.correct_point_signs(run.N, run.tab, dense)
    pts = wl.points.ravel()
    phi = wl.phi.clone()
    phi[2:] = torch.from_numpy(dense[pts].reshape(-1, 64).astype(npd)).cuda()
    assert sg.correct_package_signs(wl.grid, phi) == ref_rounds
    got, want = phi[2:].cpu().numpy().ravel(), ref[pts].astype(npd)
    assert np.array_equal(got, want) and np.array_equal(np.signbit(got), np.signbit(want))
