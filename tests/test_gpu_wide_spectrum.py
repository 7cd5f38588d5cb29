"""The z k-space pass of long lines where the spectrum or the kernel octant is past 2 GiB (the
padded sizes are asked for, so that the grids stay small): the field of every cell against the
oracle's direct sum, with planes that fill half of the z line and with two."""
import pytest

import oracle
from synthetic import random_unit_m
from tests.gpu_util import problem, rel_max, to_np

mmag = pytest.importorskip("paper_1501_07293_amd")
pytestmark = pytest.mark.gpu

CELL = 4e-9
# transforms of up to 2^29 points, 29 levels of some eps / 2 each, on the spectrum and its product
TOL = {"f32": 4e-6, "f64": 4e-14}
# spectrum of 3 nz hx Py entries past 2 GiB (8 or 16 bytes each), octant below
SPECTRUM = [("f32", (8, 8, 64), (1024, 2744, 128)), ("f32", (8, 7, 128), (1024, 1372, 256)),
            ("f32", (4, 4, 256), (512, 1400, 512)), ("f32", (4, 3, 512), (512, 700, 1024)),
            ("f64", (8, 8, 64), (1024, 1400, 128)), ("f64", (7, 8, 128), (1024, 700, 256)),
            ("f64", (4, 4, 256), (512, 700, 512))]
# octant of 6 (Pz/2+1) hx (Py/2+1) entries past 2 GiB, spectrum below
OCTANT = [("f32", (8, 8, 2), (2048, 2048, 256)), ("f32", (8, 8, 2), (1024, 2048, 512)),
          ("f32", (5, 3, 3), (1024, 1024, 1024)), ("f64", (8, 8, 2), (2048, 2240, 128)),
          ("f64", (8, 8, 2), (1024, 2048, 256)), ("f64", (8, 8, 2), (1024, 1024, 512))]


@pytest.mark.parametrize("precision,dims,pad", SPECTRUM + OCTANT)
def test_field(precision, dims, pad):
    nx, ny, nz = dims
    esz = 4 if precision == "f32" else 8
    hx = pad[0] // 2 + 1
    spectrum, octant = 3 * nz * hx * pad[1] * 2 * esz, 6 * (pad[2] // 2 + 1) * hx * (pad[1] // 2 + 1) * esz
    assert max(spectrum, octant) >= 2 ** 31
    sim = mmag.Sim(*dims, CELL, Ku=500.0, precision=precision, pad=pad)
    sim.set_m(random_unit_m((3, nz, ny, nx), seed=nz))
    ref = oracle.heff_terms(problem(*dims, CELL, Ku=500.0), to_np(sim.get_m()))["demag"]
    assert rel_max(to_np(sim.field("demag")), ref) <= TOL[precision]
    sim.close()
