"""The reverse sweep's line passes at the edges of their tiles (extents around 56 and 64 sites, columns
that do not fill a group, single sites), and the self-interaction's derivative on both sides of the
short series, against the oracle differentiated by torch autograd."""
import numpy as np
import pytest
import torch

import qlg_inputs as qi
from oracle import qlg_oracle as O
from paper_1907_12834_amd.autograd import qlg_objective
from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu

G = (1.1, -0.6, 0.8)
# three steps of up to 12 substeps, forward and back, of about 100 roundings each
TOL = {"c128": 3 * 24 * 100 * 2.0 ** -53, "c64": 3 * 24 * 100 * 2.0 ** -24}


def _oracle(psi, eps, nsteps):
    p = torch.from_numpy(psi).clone().requires_grad_(True)
    g = torch.tensor(G, dtype=torch.float64, requires_grad=True)
    a, b = O.encode(p)
    a, b = O.run(a, b, nsteps, eps, (g[0], g[1], g[2]), psi.ndim - 1)
    L = O.energy(a + b, eps, (g[0], g[1], g[2]))
    L.backward()
    return float(L.detach()), p.grad.numpy(), g.grad.numpy()


def _gpu(psi, eps, nsteps, K, dtype):
    p = torch.from_numpy(psi).to("cuda:0", torch.complex64 if dtype == "c64" else torch.complex128).requires_grad_(True)
    g = torch.tensor(G, dtype=torch.float64, requires_grad=True)
    L = qlg_objective(p, g, eps=eps, nsteps=nsteps, checkpoint_every=K, dtype=dtype)
    L.backward()
    return float(L.detach()), p.grad.cpu().numpy().astype(np.complex128), g.grad.numpy()


def _check(psi, eps, nsteps, K, dtype):
    want, got = _oracle(psi, eps, nsteps), _gpu(psi, eps, nsteps, K, dtype)
    assert abs(got[0] - want[0]) <= TOL[dtype] * abs(want[0])
    assert rel_l2(got[1], want[1]) <= TOL[dtype]
    assert rel_l2(got[2], want[2]) <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("shape", [(56,), (121,), (1, 57), (64, 3), (57, 9), (113, 2), (5, 58, 3), (59, 2, 5), (1, 1, 7)],
                         ids=str)
def test_tile_edges(shape, dtype):
    psi = qi.random_field(shape, seed=61, scale=0.4).astype(np.complex64).astype(np.complex128)
    _check(psi, 0.3, 3, 2, dtype)   # two segments, the second of one step


@pytest.mark.parametrize("eps,scale", [(0.1, 0.3), (0.5, 0.35), (1.0, 0.6)])
def test_angles(eps, scale):
    """Angles below, across and above the short series' bound, F along z on part of the lattice."""
    psi = qi.random_field((9, 70), seed=62, scale=scale)
    psi[:, :, :20] *= np.linspace(0.01, 1.0, 20)
    psi[1:4, :, 40:50] = 0.0
    _check(psi, eps, 2, 2, "c128")


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("shape", [(9, 48), (7, 49), (40, 5), (20, 7, 49), (7, 49, 5), (100, 3, 6)], ids=str)
def test_lines_laid_end_to_end(shape, dtype):
    """Windows that hold the ends of two or more lines along x, y and z."""
    psi = qi.random_field(shape, seed=63, scale=0.4).astype(np.complex64).astype(np.complex128)
    _check(psi, 0.3, 3, 2, dtype)


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("shape", [(1, 150), (2, 77), (7, 33), (24, 17), (1, 2, 50), (2, 1, 41)], ids=str)
def test_short_lines_of_several_columns(shape, dtype):
    """Runs of more than one column group along y and z, the last one with columns past the lattice."""
    psi = qi.random_field(shape, seed=64, scale=0.4).astype(np.complex64).astype(np.complex128)
    _check(psi, 0.3, 3, 2, dtype)
