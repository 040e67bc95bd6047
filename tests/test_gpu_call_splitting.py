"""A run's numbers do not depend on how it is divided into calls, nor a site's on the tile or the batch it
lies in."""
import numpy as np
import pytest
import torch

import qlg_inputs as qi
from paper_1907_12834_amd.qlg import Lattice

pytestmark = pytest.mark.gpu

G = (1.1, -0.6, 0.8)
# angles below, across and above the bound up to which a site takes the short series
ANGLES = [(0.1, 0.4), (0.3, 0.4), (0.8, 0.6)]


def _lattice(shape, dtype, qubits, eps=0.3):
    nd = len(shape)
    lat = Lattice(nd, [shape[-1]], [shape[-2]] if nd > 1 else None, [shape[0]] if nd == 3 else None, g=G, eps=eps,
                  dtype=dtype)
    lat.set_qubits([qubits])
    return lat


def _qubits(shape, scale=0.4):
    return torch.from_numpy(np.stack(qi.random_qubits(shape, seed=83, scale=scale)))


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("eps,scale", ANGLES)
@pytest.mark.parametrize("shape", [(300,), (5000,), (70000,), (40, 70), (300, 311), (10, 12, 70), (60, 64, 70)], ids=str)
def test_default_plan_resumes_bit_for_bit(shape, eps, scale, dtype):
    """A run in one call, in two, step by step, and split over two contexts."""
    q = _qubits(shape, scale)
    ref = _lattice(shape, dtype, q, eps)
    ref.step(9)
    want = ref.get_qubits()[0].cpu().numpy()
    for calls in ((5, 4), (1,) * 9):
        lat = _lattice(shape, dtype, q, eps)
        for n in calls:
            lat.step(n)
        assert np.array_equal(lat.get_qubits()[0].cpu().numpy(), want), calls
    first = _lattice(shape, dtype, q, eps)
    first.step(4)
    second = _lattice(shape, dtype, first.get_qubits()[0], eps)
    second.step(5)
    assert np.array_equal(second.get_qubits()[0].cpu().numpy(), want)


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("eps,scale", ANGLES)
@pytest.mark.parametrize("shape,plans", [
    ((300,), [{}, {"steps_per_pass": 1, "qubit_split": 2}, {"steps_per_pass": 2, "qubit_split": 2}]),
    ((300,), [{"steps_per_pass": s, "qubit_split": 0} for s in (1, 4, 7)]),
    ((300,), [{"steps_per_pass": s, "qubit_split": 1} for s in (1, 2, 7)]),
    ((40, 70), [{}] + [{"tile_rows": r, "qubit_split": q} for r, q in ((8, 0), (32, 0), (16, 1))]),
    ((10, 12, 70), [{}] + [{"tile_rows": r, "qubit_split": q} for r, q in ((8, 0), (32, 0), (16, 1))]),
], ids=["1d-2", "1d-0", "1d-1", "2d", "3d"])
def test_plans_agree_bit_for_bit(shape, plans, eps, scale, dtype):
    """Every plan does the same operations on a site in the same order (in 1D: of one qubit_split, since two
    lanes or wavefronts per site collide before the self-interaction, one lane after it)."""
    q = _qubits(shape, scale)
    out = []
    for plan in plans:
        lat = _lattice(shape, dtype, q, eps)
        if plan:
            lat.set_tuning(**plan)
        lat.step(7)
        out.append(lat.get_qubits()[0].cpu().numpy())
    for plan, x in zip(plans[1:], out[1:]):
        assert np.array_equal(x, out[0]), plan
