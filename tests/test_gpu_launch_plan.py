"""A plan that is set is the plan that runs, whatever ran before and whatever the defaults report;
use_graph alone keeps what runs; a plan of line passes reports the bands beside it."""
import ctypes

import pytest
import torch

import qlg_inputs as qi
from paper_1907_12834_amd.qlg import Lattice, Tuning, lib

pytestmark = pytest.mark.gpu

G = (1.0, -0.5, 0.5)


def _lattice(shape, dtype="c128"):
    nd = len(shape)
    lat = Lattice(nd, [shape[-1]], [shape[-2]] if nd > 1 else None, [shape[0]] if nd == 3 else None, g=G, eps=0.3,
                  dtype=dtype)
    lat.set_psi([torch.from_numpy(qi.random_field(shape, seed=7, scale=0.4))])
    return lat


def _runs(lat, **plan):
    got = lat.plan()
    return all(got[k] == v for k, v in plan.items()) and not got["line_passes"] and not got["by_size"]


@pytest.mark.parametrize("n", [97, 130, 437, 5000])
def test_one_step_per_pass_is_launched_per_step(n):
    """The defaults' own values, set on a fresh 1D lattice: three steps are three launches."""
    lat = _lattice((n,))
    lat.set_tuning(steps_per_pass=1, qubit_split=0)
    lat.set_timing(True)
    lat.step(3)
    assert lat.last_kernel_ms()[1] == 3


@pytest.mark.parametrize("shape,plan", [
    ((97,), {"steps_per_pass": 1, "qubit_split": 0}), ((97,), {"qubit_split": 0}), ((300,), {"steps_per_pass": 1}),
    ((97,), {"steps_per_pass": 3, "qubit_split": 2}), ((97,), {"qubit_split": 1}),
    ((9, 70), {"tile_rows": 32, "qubit_split": 0}), ((9, 70), {"tile_rows": 32}), ((9, 70), {"qubit_split": 0}),
    ((9, 70), {"tile_rows": 8, "qubit_split": 0}), ((9, 70), {"tile_rows": 32, "qubit_split": 1}),
    ((5, 9, 70), {"tile_rows": 32, "qubit_split": 0}), ((5, 9, 70), {"tile_rows": 8}),
])
def test_explicit_plan_runs(shape, plan):
    lat = _lattice(shape)
    assert lat.plan()["by_size"] == 1
    want = {**lat.tuning(), **plan}
    lat.set_tuning(**plan)
    assert _runs(lat, **plan) and lat.tuning() == want
    # again after another plan, and with the graph switched: the same
    lat.set_tuning(**({"steps_per_pass": 2, "qubit_split": 0} if len(shape) == 1 else {"tile_rows": 16}))
    lat.set_tuning(**plan)
    lat.set_tuning(use_graph=True)
    assert _runs(lat, use_graph=1, **plan)


@pytest.mark.parametrize("shape", [(97,), (20, 30), (6, 10, 20), (1900, 1900)])
def test_graph_alone_keeps_what_runs(shape):
    lat = _lattice(shape)
    before = lat.plan()
    lat.set_tuning(use_graph=True)
    assert lat.plan() == {**before, "use_graph": 1} and lat.plan()["by_size"] == 1
    assert lat.plan()["line_passes"] == (1 if len(shape) > 1 and shape != (1900, 1900) else 0)
    lat.set_tuning(use_graph=False)
    assert lat.plan() == before


@pytest.mark.parametrize("shape", [(48, 52), (8, 20, 24)])
def test_tuned_line_passes_do_not_stand_in_for_bands(shape, tmp_path, monkeypatch):
    """On these sizes the autotuner keeps line passes; what it reports, set on the context or on a new
    one of the size class, runs as bands, eight rows too."""
    monkeypatch.setenv("QLG_TUNE_CACHE", str(tmp_path / "tune.txt"))
    lat = _lattice(shape)
    plan = lat.autotune()
    assert lat.plan()["line_passes"] == 1 and lat.plan()["by_size"] == 0
    lat.set_tuning(use_graph=True)
    assert lat.plan()["line_passes"] == 1
    other = _lattice(shape)
    assert other.plan()["line_passes"] == 1 and other.tuning() == plan
    other.set_tuning(tile_rows=8, qubit_split=0)
    assert _runs(other, tile_rows=8, qubit_split=0)
    t = Tuning()   # the C calls: read, change the graph, set
    assert lib().qlg_get_tuning(lat.ctx, ctypes.byref(t)) == 0
    t.use_graph = 0
    assert lib().qlg_set_tuning(lat.ctx, ctypes.byref(t)) == 0
    assert _runs(lat, **plan)
