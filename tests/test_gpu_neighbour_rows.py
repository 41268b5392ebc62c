"""The neighbour table where a row of three cells does not fit the grid or ends
at its faces: grids of one to five cells a side and of 33, with every cell
activated, none, and some of those at the faces, against the oracle bit for
bit."""
import numpy as np
import pytest
import torch

import oracle
from tables_check import assert_tables_equal

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("field", ["all", "none", "some"])
@pytest.mark.parametrize("M", [1, 2, 3, 4, 5, 33])
def test_neighbour_rows_match_oracle(M, field):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2512_11473_amd as sg
    d = np.full(M ** 3, -9.0, dtype=np.float32)
    if field == "all":
        d[:] = 0.0
    elif field == "some":
        rng = np.random.default_rng(M)
        faces = np.arange(M ** 3)
        at_face = np.zeros(M ** 3, dtype=bool)
        for c in (faces % M, (faces // M) % M, faces // (M * M)):
            at_face |= (c == 0) | (c == M - 1)
        on = np.nonzero(at_face)[0]
        d[rng.choice(on, size=max(1, len(on) // 20), replace=False)] = 0.0
    ref = oracle.build_tables(M, d)
    g = sg.build_packages(torch.from_numpy(d).cuda(), 1.0 / (4 * M))
    assert_tables_equal({k: v.cpu().numpy() for k, v in g.tables().items()}, ref)
