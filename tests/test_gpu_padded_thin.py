"""One-cell-thick grids with a padded z axis (six kernel spectra, transformed along z too):
RK4 and Euler steps against the separate passes, the unpadded grid and the oracle, on grids
small enough for one work-group and past that."""
import numpy as np
import pytest

import oracle
from synthetic import random_unit_m
from tests.gpu_util import problem, rel_max, to_np

mmag = pytest.importorskip("paper_1501_07293_amd")
pytestmark = pytest.mark.gpu

CELL = 4e-9
# as the unpadded grids': 5 x 4 stages, 0.1 of a unit per unit of the field, 30 eps of it each
TOL = {"f32": 8e-6, "f64": 2e-14}


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("pz", [2, 3, 4, 6])
@pytest.mark.parametrize("dims", [(16, 8, 1), (8, 8, 1), (1, 1, 1), (40, 30, 1)])
def test_steps(dims, pz, precision):
    nx, ny, nz = dims
    m0 = random_unit_m((3, nz, ny, nx), seed=nx + pz)
    out = []
    for kw in (dict(pad=(0, 0, pz)), dict(pad=(0, 0, pz), split_stage=True), dict()):
        sim = mmag.Sim(*dims, CELL, Ku=2e4, alpha=0.3, precision=precision, **kw)
        sim.set_m(m0)
        sim.set_hext((1e4, -2e4, 3e4))
        m_used = to_np(sim.get_m())
        sim.step(3, 1e-13)
        out.append(to_np(sim.get_m()))
        sim.step_euler(2, 1e-14)
        out.append(to_np(sim.get_m()))
    for a, b in ((0, 2), (1, 3), (0, 4), (1, 5)):
        assert rel_max(out[a], out[b]) <= TOL[precision]
    pb = problem(*dims, CELL, Ku=2e4, alpha=0.3, hext=(1e4, -2e4, 3e4))
    assert np.abs(out[0] - oracle.rk4(pb, m_used, 1e-13, 3)).max() <= (2e-5 if precision == "f32" else 1e-11)
