"""Line passes (one launch per axis, small 2D and 3D lattices in the default plan) at the edges of
their tiles: extents of one site, around 56 and 64 sites, around the columns of a group and the rows
of an x tile, batches, with a potential, in both splits and dtypes, against the oracle; and against
bands, graph replays and saved plans."""
import numpy as np
import pytest
import torch

import qlg_inputs as qi
from oracle import qlg_oracle as O
from paper_1907_12834_amd.qlg import Lattice
from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu

G = (1.0, -0.5, 0.5)


def _lattice(shapes, dtype, split="interleaved"):
    nd = len(shapes[0])
    return Lattice(nd, [s[-1] for s in shapes], [s[-2] for s in shapes], [s[0] for s in shapes] if nd == 3 else None,
                   g=G, eps=0.3, dtype=dtype, split=split)


def _qubits(shapes, seed):
    return [np.stack(qi.random_qubits(sh, seed=seed + i, scale=0.4)) for i, sh in enumerate(shapes)]


def _oracle(q, n, split, V=None, mu=0.0):
    a, b = O.run(torch.from_numpy(q[0]), torch.from_numpy(q[1]), n, 0.3, G, q.ndim - 2, split, V=V, mu=mu)
    return np.stack([a.numpy(), b.numpy()])


SHAPES = [[(1, 1)], [(7, 3), (9, 5), (1, 130)], [(56, 64), (57, 57)], [(64, 56), (121, 9)], [(130, 1), (8, 66)],
          [(1, 1, 1), (2, 57, 3)], [(57, 8, 5), (3, 9, 60)], [(13, 64, 9)]]


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("split", ["interleaved", "plain"])
@pytest.mark.parametrize("shapes", SHAPES, ids=str)
def test_line_passes_match_oracle(shapes, split, dtype):
    qs = _qubits(shapes, 90)
    lat = _lattice(shapes, dtype, split)
    lat.set_qubits([torch.from_numpy(q) for q in qs])
    lat.step(1)      # the step that records the overlap
    lat.step(3)      # two that do not, then one that does
    for q, got in zip(qs, lat.get_qubits()):
        assert rel_l2(got.cpu().numpy(), _oracle(q, 4, split)) <= (1e-12 if dtype == "c128" else 1e-5)


@pytest.mark.parametrize("shape", [(70, 59), (9, 17, 58)])
def test_line_passes_with_potential_and_overlap(shape):
    """(V + mu) phase of every line kernel, and the overlap energy of the last step."""
    q = _qubits([shape], 95)[0]
    V = np.random.default_rng(4).normal(size=shape)
    lat = _lattice([shape], "c128")
    lat.set_potential([torch.from_numpy(V)], 0.3)
    lat.set_qubits([torch.from_numpy(q)])
    lat.step(3)
    ref = _oracle(q, 3, "interleaved", V, 0.3)
    assert rel_l2(lat.get_qubits()[0].cpu().numpy(), ref) <= 1e-12
    prev = _oracle(q, 2, "interleaved", V, 0.3)
    o = lat.observables()[0]
    ov = 0.3 ** len(shape) * np.vdot(ref[0] + ref[1], prev[0] + prev[1])
    assert abs(o["overlap"] - ov) <= 1e-12 * abs(ov)


@pytest.mark.parametrize("shapes", [[(66, 120), (20, 31)], [(10, 12, 70), (60, 5, 9)]], ids=str)
@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_forms_give_the_same_numbers(shapes, dtype):
    """Default form, bands and replayed graphs, from a run that changes plan between calls."""
    qs = [torch.from_numpy(q) for q in _qubits(shapes, 97)]
    out = []
    for plan in (None, {"use_graph": True}, {"tile_rows": 16}, {"tile_rows": 8, "qubit_split": 1, "use_graph": True}):
        lat = _lattice(shapes, dtype)
        lat.set_qubits(qs)
        lat.step(2)
        if plan:
            lat.set_tuning(**plan)
        for n in (1, 4, 5, 4, 5):
            lat.step(n)
        out.append([x.cpu().numpy() for x in lat.get_qubits()])
    for other in out[1:]:
        for x, y in zip(out[0], other):
            assert rel_l2(x, y) <= (1e-13 if dtype == "c128" else 2e-6)
    for x, y in zip(out[0], out[1]):
        assert np.array_equal(x, y)


def test_saved_plan_of_line_passes(tmp_path, monkeypatch):
    """A '|lines' entry of the plan file gives the default form's numbers, a later entry of the bare key bands."""
    monkeypatch.setenv("QLG_TUNE_CACHE", str(tmp_path / "tune.txt"))
    key = "%s|1|2|0|0|%d" % (torch.cuda.get_device_properties(0).gcnArchName, (40 * 50 - 1).bit_length())
    q = [torch.from_numpy(x) for x in _qubits([(40, 50)], 99)]
    out = []
    for text in ("", "%s|lines 1 8 1 0\n" % key, "%s|lines 1 8 1 0\n%s 1 24 0 1\n" % (key, key)):
        (tmp_path / "tune.txt").write_text(text)
        lat = _lattice([(40, 50)], "c128")
        out.append((lat.tuning(), lat))
        lat.set_qubits(q)
        lat.step(6)
    assert out[1][0] == {"steps_per_pass": 1, "tile_rows": 8, "use_graph": 1, "qubit_split": 0}
    assert out[2][0] == {"steps_per_pass": 1, "tile_rows": 24, "use_graph": 0, "qubit_split": 1}
    a, b, c = (x[1].get_qubits()[0].cpu().numpy() for x in out)
    assert np.array_equal(a, b) and rel_l2(c, a) <= 1e-13


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("shapes", [[(11, 47), (9, 48), (10, 49)], [(300, 4)], [(31, 70), (1, 104), (25, 105)],
                                    [(5, 49, 20), (20, 5, 49)], [(49, 20, 3), (9, 100, 4)], [(100, 7, 9)], [(6, 21, 2)]], ids=str)
def test_lines_laid_end_to_end(shapes, dtype):
    """Windows that hold the ends of two lines, of many short ones, or (48, 104 sites: as many slots
    either way; 49, 105: fewer end to end) begin with each line; and the overlap of the last step."""
    qs = _qubits(shapes, 101)
    lat = _lattice(shapes, dtype)
    lat.set_qubits([torch.from_numpy(q) for q in qs])
    lat.step(3)
    tol = 1e-12 if dtype == "c128" else 1e-5
    for q, got, o in zip(qs, lat.get_qubits(), lat.observables()):
        ref, prev = _oracle(q, 3, "interleaved"), _oracle(q, 2, "interleaved")
        assert rel_l2(got.cpu().numpy(), ref) <= tol
        ov = 0.3 ** (q.ndim - 2) * np.vdot(ref[0] + ref[1], prev[0] + prev[1])
        assert abs(o["overlap"] - ov) <= tol * abs(ov)


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("shapes", [[(2, 150), (7, 77), (24, 9)], [(1, 2, 61), (2, 1, 41), (3, 2, 30)]], ids=str)
def test_short_lines_of_several_columns(shapes, dtype):
    """Runs of more than one column group along y and z, with a potential."""
    qs = _qubits(shapes, 111)
    Vs = [np.random.default_rng(5 + i).normal(size=s) for i, s in enumerate(shapes)]
    lat = _lattice(shapes, dtype)
    lat.set_potential([torch.from_numpy(V) for V in Vs], 0.2)
    lat.set_qubits([torch.from_numpy(q) for q in qs])
    lat.step(3)
    for q, V, got in zip(qs, Vs, lat.get_qubits()):
        assert rel_l2(got.cpu().numpy(), _oracle(q, 3, "interleaved", V, 0.2)) <= (1e-12 if dtype == "c128" else 1e-5)
