"""The ordered core list at the edges of its partitions: chunks of 256 sites, four of them per counting
and eight per writing wavefront, 16384 per turn of the scan; dense and sparse cores, a list cut off
at its capacity.  Integers, so they agree exactly with the windings of the vorticity output."""
import numpy as np
import pytest
import torch

from paper_1907_12834_amd.qlg import Lattice, lib

pytestmark = pytest.mark.gpu


def _lattice(shapes, dense):
    nd = len(shapes[0])
    lat = Lattice(nd, [s[-1] for s in shapes], [s[-2] for s in shapes], [s[0] for s in shapes] if nd == 3 else None,
                  g=(1.0, 0.0, 0.0), eps=0.5, dtype="c64")
    gen = torch.Generator(device="cuda").manual_seed(7)
    psis = []
    for sh in shapes:
        p = torch.randn((5,) + sh, dtype=torch.complex64, device="cuda", generator=gen)
        if not dense:   # a uniform phase but for a few sites
            keep = torch.rand(sh, device="cuda", generator=gen) < 2e-4
            keep.view(-1)[-1] = keep.view(-1)[0] = True
            p = torch.where(keep, p, torch.ones_like(p))
        psis.append(p)
    lat.set_psi(psis)
    return lat


def _expected(lat, shapes):
    rows = []
    for i, (sh, v) in enumerate(zip(shapes, lat.vorticity(0))):
        w = v["winding"].cpu().numpy()
        at = np.argwhere(w != 0)
        one = np.column_stack([np.full(len(at), i), at, w[w != 0]])
        rows.append(one)
    rows = np.concatenate(rows)
    if len(shapes[0]) == 3:   # family first
        rows = rows[np.argsort(rows[:, 1], kind="stable")]
    return rows


@pytest.mark.parametrize("dense", [True, False])
@pytest.mark.parametrize("shapes", [[(1, 1)], [(16, 16), (257, 1), (15, 17)], [(16, 65), (16, 64), (16, 63)], [(131, 257)],
                                    [(2048, 2048)], [(2049, 2049)], [(5, 7, 9), (31, 8, 33)]], ids=str)
def test_core_list(shapes, dense):
    lat = _lattice(shapes, dense)
    want = _expected(lat, shapes)
    got = lat.find_vortices(0)
    assert np.array_equal(got.cpu().numpy(), want)
    # cut off at a capacity: the list's start, nothing after it, and the true count
    cap, n = max(len(want) // 3, 1), torch.zeros(1, dtype=torch.int64, device="cuda")
    sites = sum(int(np.prod(s)) for s in shapes) * (3 if len(shapes[0]) == 3 else 1)
    wind = torch.empty(sites, dtype=torch.int32, device="cuda")
    cores = torch.full((cap + 4, want.shape[1]), -7, dtype=torch.int32, device="cuda")
    assert lib().qlg_find_vortices(lat.ctx, 0, wind.data_ptr(), cores.data_ptr(), cap, n.data_ptr()) == 0
    assert int(n.item()) == len(want)
    assert np.array_equal(cores[:min(cap, len(want))].cpu().numpy(), want[:cap])
    assert (cores[cap:] == -7).all()
