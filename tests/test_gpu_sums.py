"""Sums over a lattice at the edges of their partitions: wavefronts of 64 and chunks of 256 sites, the
960 threads that add the chunks' partial sums, and the overlap partials of bands and line passes."""
import numpy as np
import pytest
import torch

import qlg_inputs as qi
from oracle import qlg_oracle as O
from paper_1907_12834_amd.qlg import Lattice

pytestmark = pytest.mark.gpu

G = (1.0, -0.4, 0.3)
EPS = 0.2


@pytest.mark.parametrize("shapes", [[(1,)], [(63,), (64,), (65,), (257,)], [(96 * 256,)], [(96 * 256 + 1,)],
                                    [(481 * 56 + 3,)], [(56, 64), (481, 9)], [(3, 40, 60)]], ids=str)
def test_observables_match_oracle(shapes):
    nd = len(shapes[0])
    qs = [np.stack(qi.random_qubits(sh, seed=120 + i, scale=0.4)) for i, sh in enumerate(shapes)]
    lat = Lattice(nd, [s[-1] for s in shapes], [s[-2] for s in shapes] if nd > 1 else None,
                  [s[0] for s in shapes] if nd == 3 else None, g=G, eps=EPS, dtype="c128")
    lat.set_qubits([torch.from_numpy(q) for q in qs])
    lat.step(1)
    for q, o in zip(qs, lat.observables()):
        a0, b0 = torch.from_numpy(q[0]), torch.from_numpy(q[1])
        a, b = O.run(a0, b0, 1, EPS, G, nd)
        psi, prev = (a + b).numpy(), (a0 + b0).numpy()
        w = EPS ** nd
        # one step of 4 to 12 substeps of about 100 roundings, on sums of positive terms
        tol = 12 * 100 * 2.0 ** -53
        n = w * np.sum(np.abs(psi) ** 2)
        assert abs(o["norm_psi"] - n) <= tol * n
        assert np.allclose(o["pop"], w * (np.abs(psi) ** 2).reshape(5, -1).sum(1), rtol=tol, atol=tol * n)
        ov = w * np.vdot(psi, prev)
        assert abs(o["overlap"] - ov) <= tol * w * np.linalg.norm(psi) * np.linalg.norm(prev)
        e, scale = float(O.energy(a + b, EPS, G)), float(O.energy(a + b, EPS, [abs(g) for g in G]))
        assert abs(o["energy"] - e) <= 4 * tol * scale
