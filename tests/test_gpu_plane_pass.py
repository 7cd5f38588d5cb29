"""The plane pass (y forward, z k-space and y inverse of an x bin in one work-group, z lines
in registers): every z length it serves, open and periodic, with the planes on either side
of the size where it hands over to separate passes, against the oracle's field."""
import pytest

import oracle
from tests.gpu_util import problem, rel_max, to_np
from synthetic import random_unit_m

mmag = pytest.importorskip("paper_1501_07293_amd")
pytestmark = pytest.mark.gpu

CELL = 4e-9
# FFTs over up to 2^13 points of data rounded to the working precision: some 30 eps on the
# largest field entry
TOL = {"f32": 2e-6, "f64": 2e-14}


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("Pz", [3, 4, 5, 6, 7, 8, 9, 10, 12])
@pytest.mark.parametrize("ny", [1, 2, 7, 61, 128, 250, 520])
def test_open(Pz, ny, precision):
    # rows of one to three y stages, one round of columns (threads to spare) and two; the
    # last is past the hand-over at every Pz
    nz = (Pz + 1) // 2
    sim = mmag.Sim(4, ny, nz, CELL, Ku=500.0, precision=precision, pad=(0, 0, Pz))
    assert sim.plan()["pz"] == Pz
    sim.set_m(random_unit_m((3, nz, ny, 4), seed=ny + Pz))
    ref = oracle.heff_terms(problem(4, ny, nz, CELL, Ku=500.0), to_np(sim.get_m()))["demag"]
    assert rel_max(to_np(sim.field("demag")), ref) <= TOL[precision]


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("dims,periodic", [((6, 9, 5), (True, True, False)), ((5, 12, 8), (False, False, True)),
                                           ((9, 10, 7), (True, True, True)), ((7, 3, 3), (False, True, True))])
def test_periodic_matches_runtime_passes(dims, periodic, precision):
    # along a periodic axis the line is the grid's own length: nz = Pz, odd rows
    out = []
    for generic in (False, True):
        sim = mmag.Sim(*dims, CELL, Ku=500.0, precision=precision, periodic=periodic, generic_fft=generic)
        sim.set_m(random_unit_m((3, dims[2], dims[1], dims[0]), seed=3))
        out.append(to_np(sim.field("demag")))
    assert rel_max(out[0], out[1]) <= 2 * TOL[precision]
