"""The ordered core list where a wavefront takes one, two and several chunks (2048 chunks and one more) and
the scan one count per thread and several (1024 and one more; three plane families in 3D), lists cut off,
a NULL list of no capacity."""
import numpy as np
import pytest
import torch

from paper_1907_12834_amd.qlg import lib
from tests.test_gpu_cores import _expected, _lattice

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dense", [True, False])
@pytest.mark.parametrize("shapes", [[(1024, 256)], [(1025, 256)], [(2048, 256)], [(2049, 256)], [(16, 16), (4097, 256)], [(60, 51, 57)], [(683, 16, 16)],
                                    [(100, 101, 99)]], ids=str)
def test_core_list(shapes, dense):
    lat = _lattice(shapes, dense)
    want = _expected(lat, shapes)
    assert np.array_equal(lat.find_vortices(0, capacity=len(want) + 5).cpu().numpy(), want)
    sites = sum(int(np.prod(s)) for s in shapes) * (3 if len(shapes[0]) == 3 else 1)
    wind = torch.empty(sites, dtype=torch.int32, device="cuda")
    n = torch.zeros(1, dtype=torch.int64, device="cuda")
    for cap in (0, max(len(want) // 2, 1)):
        cores = torch.full((cap + 4, want.shape[1]), -7, dtype=torch.int32, device="cuda")
        assert lib().qlg_find_vortices(lat.ctx, 0, wind.data_ptr(), cores.data_ptr() if cap else None, cap, n.data_ptr()) == 0
        assert int(n.item()) == len(want)
        assert np.array_equal(cores[:min(cap, len(want))].cpu().numpy(), want[:cap]) and (cores[cap:] == -7).all()
