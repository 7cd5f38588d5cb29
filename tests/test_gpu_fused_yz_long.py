"""The fused y-z pass where a work-group's threads hold only one z line a round (FP64 lines of
1029 points, 343 threads each), two (FP32) and several, against the separate passes and the oracle."""
import numpy as np
import pytest

import oracle
from synthetic import random_unit_m
from tests.gpu_util import problem, rel_max, to_np

mmag = pytest.importorskip("paper_1501_07293_amd")
pytestmark = pytest.mark.gpu

CELL = 4e-9
# FFTs over up to 2^13 points of data rounded to the working precision: some 30 eps on the
# largest field entry
TOL = {"f32": 2e-6, "f64": 2e-14}


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("dims,periodic_z", [((2, 1, 515), False), ((3, 1, 513), False), ((2, 1, 1029), True),
                                             ((2, 1, 500), False), ((2, 2, 343), True)])
def test_field(dims, periodic_z, precision):
    nx, ny, nz = dims
    out = []
    for fused in (True, False):
        sim = mmag.Sim(*dims, CELL, Ku=500.0, precision=precision, fused_yz=fused, threads=512,
                       periodic=(False, False, periodic_z))
        assert sim.plan()["passes"] == (3 if fused else 5)
        sim.set_m(random_unit_m((3, nz, ny, nx), seed=nz))
        out.append(to_np(sim.field("demag")))
    assert rel_max(out[0], out[1]) <= 2 * TOL[precision]
    if not periodic_z:
        ref = oracle.heff_terms(problem(*dims, CELL, Ku=500.0), to_np(sim.get_m()))["demag"]
        assert rel_max(out[0], ref) <= TOL[precision]
