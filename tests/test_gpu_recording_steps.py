"""Steps that record the overlap: in 3D line passes run their y and x axes as bands, and 1D passes of fewer
steps than the plan's use part of its tiles."""
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


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("sizes", [[300], [33000], [70001], [8, 24, 25, 56, 57, 97, 130], [1, 40000, 3]], ids=str)
@pytest.mark.parametrize("plan", [{}, {"steps_per_pass": 7, "qubit_split": 0}, {"steps_per_pass": 3, "qubit_split": 2},
                                  {"steps_per_pass": 5, "qubit_split": 1}], ids=str)
def test_overlap_of_passes_of_fewer_steps(plan, sizes, dtype):
    """1D passes of fewer steps than the plan's leave tiles of the table empty: the overlap of each length
    of pass, after one of another length, against the two states."""
    lat = Lattice(1, sizes, g=G, eps=0.3, dtype=dtype)
    lat.set_qubits([_qubits((n,)) for n in sizes])
    if plan:
        lat.set_tuning(**plan)
    twin = Lattice(1, sizes, g=G, eps=0.3, dtype=dtype)
    twin.set_qubits([_qubits((n,)) for n in sizes])
    for n in (7, 1, 2, 4, 3, 1):
        twin.step(n - 1)
        prev = [x.cpu().to(torch.complex128).sum(0).numpy() for x in twin.get_qubits()]
        twin.step(1)
        lat.step(n)
        for x, p, o in zip(lat.get_qubits(), prev, lat.observables()):
            ov = 0.3 * np.vdot(x.cpu().to(torch.complex128).sum(0).numpy(), p)
            assert abs(o["overlap"] - ov) <= (1e-12 if dtype == "c128" else 1e-5) * abs(ov), n
