"""Lattices above the line passes' sizes in the plan that the library chooses (bands of the height that costs
least in rounds of tiles), nothing tuned or set: light-cone windows against the oracle."""
import numpy as np
import pytest
import torch

import qlg_inputs as qi
from paper_1907_12834_amd.qlg import Lattice
from tests.helpers import light_cone_oracle_2d, rel_l2

pytestmark = pytest.mark.gpu

G = (1.0, -0.5, 0.5)


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("ny,nx", [(1700, 1801), (2900, 1003)])
def test_untuned_large_lattice(ny, nx, dtype):
    psi = qi.random_field((ny, nx), seed=12, scale=0.4)
    lat = Lattice(2, [nx], [ny], g=G, eps=0.3, dtype=dtype)
    plan = lat.plan()
    assert plan["by_size"] == 1 and plan["line_passes"] == 0
    lat.set_psi([torch.from_numpy(psi)])
    lat.step(3)
    got = lat.get_psi()[0].cpu().numpy()
    rows = plan["tile_rows"]
    # inside a band and a tile, across their edges, the last band's end, both wraps
    for cy, cx in ((5, 30), (rows, 56), (2 * rows, 56 * 17), (ny - 1, 300), (rows * (ny // rows), 700), (900, nx - 1), (0, 0)):
        ref = light_cone_oracle_2d(psi, cy, cx, 3, 0.3, G, half_out=2)
        sub = got[:, (np.arange(cy - 2, cy + 3) % ny)[:, None], (np.arange(cx - 2, cx + 3) % nx)[None, :]]
        assert rel_l2(sub, ref) <= (1e-12 if dtype == "c128" else 1e-5), (cy, cx)
