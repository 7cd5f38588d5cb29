"""The long-line z pass over column counts around its work-group grouping: fewer work-groups
than a group on each XCD, whole groups, and remainders; against the oracle's field."""
import pytest

import oracle
from synthetic import random_unit_m
from tests.gpu_util import problem, rel_max, to_np

mmag = pytest.importorskip("paper_1501_07293_amd")
pytestmark = pytest.mark.gpu

CELL = 4e-9
# FFTs over up to 2^21 points of data rounded to the working precision: some 40 eps on the
# largest field entry
TOL = {"f32": 2.5e-6, "f64": 2.5e-14}


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("pz", [128, 256, 512])
@pytest.mark.parametrize("px,py", [(2, 2), (16, 14), (30, 32), (64, 35), (128, 64)])
def test_field(px, py, pz, precision):
    nx, ny, nz = min(px // 2, 8), min(py // 2, 6), 9
    sim = mmag.Sim(nx, ny, nz, CELL, Ku=500.0, precision=precision, pad=(px, py, pz), split_yz=True)
    assert sim.routes()["long_z"] == mmag.ZLINE_LONG
    sim.set_m(random_unit_m((3, nz, ny, nx), seed=px + py))
    ref = oracle.heff_terms(problem(nx, ny, nz, CELL, Ku=500.0), to_np(sim.get_m()))["demag"]
    assert rel_max(to_np(sim.field("demag")), ref) <= TOL[precision]
