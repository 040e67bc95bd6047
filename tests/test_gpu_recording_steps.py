"""Steps that record the overlap: in 3D line passes run their y and x axes as bands."""
import numpy as np
import pytest
import torch

import qlg_inputs as qi
from paper_1907_12834_amd.qlg import Lattice
from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu

G = (1.1, -0.6, 0.8)


def _lattice(shape, dtype, qubits, eps=0.3):
    nd = len(shape)
    lat = Lattice(nd, [shape[-1]], [shape[-2]] if nd > 1 else None, [shape[0]] if nd == 3 else None, g=G, eps=eps,
                  dtype=dtype)
    lat.set_qubits([qubits])
    return lat


def _qubits(shape, scale=0.4):
    return torch.from_numpy(np.stack(qi.random_qubits(shape, seed=83, scale=scale)))


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("shape", [(64, 120, 130), (140, 57, 60)], ids=str)
def test_recording_bands_are_tall_enough(shape, dtype):
    """With more tiles of eight rows than SIMDs the recording step's bands are taller; the same numbers."""
    q = _qubits(shape)
    lat, bands = _lattice(shape, dtype, q), _lattice(shape, dtype, q)
    assert lat.plan()["line_passes"] == 1 and lat.plan()["tile_rows"] > 8
    bands.set_tuning(tile_rows=32)
    for n in (1, 3, 1):
        lat.step(n)
        bands.step(n)
        x, y = lat.observables()[0], bands.observables()[0]
        assert abs(x["overlap"] - y["overlap"]) <= (1e-12 if dtype == "c128" else 1e-5) * abs(y["overlap"])
    assert rel_l2(lat.get_qubits()[0].cpu().numpy(), bands.get_qubits()[0].cpu().numpy()) <= (1e-13 if dtype == "c128" else 2e-6)
