"""The reverse sweep along y and z axes of one to three sites, whose windows hold whole lines as rings
of lanes: line counts around those of a window (64, 32 and 21), axes of four sites beside them, batches
that mix both, with a potential, against the oracle differentiated by torch autograd."""
import numpy as np
import pytest
import torch

import qlg_inputs as qi
from oracle import qlg_oracle as O
from paper_1907_12834_amd.qlg import Lattice
from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu

G = (1.1, -0.6, 0.8)
EPS, STEPS, MU = 0.3, 3, 0.2
# three steps of up to 12 substeps, forward and back, of about 100 roundings each
TOL = {"c128": 3 * 24 * 100 * 2.0 ** -53, "c64": 3 * 24 * 100 * 2.0 ** -24}


def _oracle(q, V):
    z = [torch.from_numpy(x).clone().requires_grad_(True) for x in q]
    g = torch.tensor(G, dtype=torch.float64, requires_grad=True)
    v = torch.from_numpy(V)
    a, b = O.run(z[0], z[1], STEPS, EPS, (g[0], g[1], g[2]), V.ndim, V=v, mu=MU)
    L = O.energy(a + b, EPS, (g[0], g[1], g[2]), V=v, mu=MU)
    L.backward()
    return float(L.detach()), np.stack([x.grad.numpy() for x in z]), g.grad.numpy()


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("shapes", [
    [(1, 1)], [(1, 63), (1, 64), (1, 65)], [(2, 31), (2, 32), (2, 33), (9, 40)], [(3, 20), (4, 21), (3, 21), (3, 22)],
    [(1, 7, 9), (2, 5, 13), (3, 3, 7), (4, 3, 8)], [(7, 1, 9), (5, 2, 13), (1, 3, 22), (6, 4, 5)],
    [(2, 3, 64), (3, 2, 43), (1, 1, 130)], [(130, 2), (3, 1), (2, 2)]], ids=str)
def test_thin_axes(shapes, dtype):
    nd = len(shapes[0])
    qs = [np.stack(qi.random_qubits(s, seed=71 + i, scale=0.4)).astype(np.complex64).astype(np.complex128)
          for i, s in enumerate(shapes)]
    Vs = [np.random.default_rng(6 + i).normal(size=s) for i, s in enumerate(shapes)]
    lat = Lattice(nd, [s[-1] for s in shapes], [s[-2] for s in shapes], [s[0] for s in shapes] if nd == 3 else None, g=G,
                  eps=EPS, dtype=dtype)
    lat.set_potential([torch.from_numpy(V) for V in Vs], MU)
    lat.set_qubits([torch.from_numpy(q) for q in qs])
    ck = lat.forward_record(STEPS, 2)   # two segments, the second of one step
    value, lam, dg = lat.objective_grad("energy")
    dg = np.array(dg) + np.array(lat.adjoint_step(STEPS, 2, ck, lam))
    want = [_oracle(q, V) for q, V in zip(qs, Vs)]
    assert abs(value - sum(w[0] for w in want)) <= TOL[dtype] * sum(abs(w[0]) for w in want)
    o, lam = 0, lam.cpu().numpy()
    for s, w in zip(shapes, want):
        n = 10 * int(np.prod(s))
        assert rel_l2(lam[o:o + n].reshape((2, 5) + s), w[1]) <= TOL[dtype], s
        o += n
    assert rel_l2(dg, sum(w[2] for w in want)) <= TOL[dtype]
