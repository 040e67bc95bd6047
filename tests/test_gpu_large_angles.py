"""Phases far beyond the short series, on the GPU against the oracle: external phases of many turns beside
small self-interaction angles."""
import numpy as np
import pytest
import torch

import qlg_inputs as qi
from oracle import qlg_oracle as O
from paper_1907_12834_amd.qlg import Lattice
from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu

G = (1.0, -0.7, 0.4)
UNIT = {"c128": 2.0 ** -53, "c64": 2.0 ** -24}


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("phase,scale", [(3.0, 0.3), (200.0, 1e-3), (20000.0, 1e-3)])
def test_many_turns(dtype, phase, scale):
    L = 203
    psi = qi.random_field((L,), seed=41, scale=scale).astype(np.complex64).astype(np.complex128)
    V = phase * np.linspace(-1.0, 1.0, L)   # sites on both sides of every line in one wavefront
    a, b = O.run_psi(psi, 1, 1.0, G, V=torch.from_numpy(V))
    lat = Lattice(1, [L], g=G, eps=1.0, dtype=dtype)
    lat.set_potential([V], 0.0)
    lat.set_psi([torch.from_numpy(psi)])
    lat.step(1)
    got = lat.get_qubits()[0].cpu().numpy()
    # four substeps of about 40 roundings each, and phases that add up to `phase`, whose own roundings
    # (about eight unit roundoffs of the phase, in either program) turn the state by as much
    assert rel_l2(got, np.stack([a.numpy(), b.numpy()])) <= UNIT[dtype] * (160 + 16 * phase)
