"""The self-interaction at its edges: rotation angles on both sides of the short series, states
whose spin vector is zero, along z or tiny, and components that stay exactly empty."""
import numpy as np
import pytest
import torch

import qlg_inputs as qi
from oracle import qlg_oracle as O
from paper_1907_12834_amd.qlg import Lattice
from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu

G = (1.0, -0.7, 0.4)
# one 1D step: four substeps of about 40 roundings each, at unit roundoff
TOL = {"c128": 160 * 2.0 ** -53, "c64": 160 * 2.0 ** -24}


def _one_step(psi, eps, dtype, split, qubit_split=0):
    lat = Lattice(1, [psi.shape[1]], g=G, eps=eps, dtype=dtype, split=split)
    lat.set_tuning(qubit_split=qubit_split)
    lat.set_psi([torch.from_numpy(psi)])
    lat.step(1)
    return lat.get_qubits()[0].cpu().numpy()


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("split,qubit_split", [("interleaved", 0), ("interleaved", 1), ("interleaved", 2), ("plain", 0)])
# eps^2 n: angles well below, across and well above the short series' bound
@pytest.mark.parametrize("eps,scale", [(0.1, 0.4), (0.5, 0.35), (1.0, 0.8), (0.1, 1e-12)])
def test_angles(dtype, split, qubit_split, eps, scale):
    psi = qi.random_field((97,), seed=31, scale=scale)
    psi[:, :20] *= np.linspace(0.01, 1.0, 20)   # both branches of a wavefront's lanes
    psi = psi.astype(np.complex64).astype(np.complex128)
    a, b = O.run_psi(psi, 1, eps, G, split)
    got = _one_step(psi, eps, dtype, split, qubit_split)
    assert rel_l2(got, np.stack([a.numpy(), b.numpy()])) <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("eps", [0.1, 1.0])
@pytest.mark.parametrize("filled", [[0], [1], [2], [4], [0, 4], [0, 2, 4], [1, 3], [0, 3]])
def test_empty_components_stay_empty(dtype, eps, filled):
    """These components are closed under the step: the others have no source."""
    psi = np.zeros((5, 130), complex)
    psi[filled] = qi.random_field((130,), seed=32, scale=0.5)[filled].astype(np.complex64)
    a, b = O.run_psi(psi, 1, eps, G)
    got = _one_step(psi, eps, dtype, "interleaved")
    assert rel_l2(got, np.stack([a.numpy(), b.numpy()])) <= TOL[dtype]
    empty = [m for m in range(5) if m not in filled]
    assert np.abs(got[:, empty]).max() == 0.0
