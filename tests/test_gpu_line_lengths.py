"""The runtime-length register passes at the lengths where a schedule changes: every
radix alone and in each position, one to five stages, odd lengths, lengths whose line
takes more threads than a work-group has, along each axis and in a batch, against the
oracle's direct sum (Eqs. 12-13)."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import problem, rel_max, to_np
from synthetic import random_unit_m

mmag = pytest.importorskip("paper_1501_07293_amd")
pytestmark = pytest.mark.gpu

CELL = 4e-9
# both sides are FFTs over up to 2^12 points of data rounded to the working precision:
# about eps per butterfly level on the largest field entry, some 30 eps in all, plus the
# FP64 rounding of the tensor and its spectrum
TOL = {"f32": 2e-6, "f64": 2e-14}

# one stage; two; three; four and five; odd lengths among each
LENGTHS = [2, 3, 4, 5, 6, 7, 8, 9, 10, 12, 14, 15, 16,
           18, 21, 25, 32, 49, 60, 64, 84, 98, 100, 128, 150, 225, 256,
           162, 250, 336, 343, 384, 405, 500, 512, 600, 625, 686, 729, 1024]
LONG = [2187, 2401, 3125, 4096, 6250]


def demag_error(dims, pad, precision, generic=True):
    sim = mmag.Sim(*dims, CELL, Ku=500.0, precision=precision, pad=pad, generic_fft=generic)
    p = sim.plan()
    for k, v in zip(("px", "py", "pz"), pad):
        assert v == 0 or p[k] == v, p
    sim.set_m(random_unit_m((3, dims[2], dims[1], dims[0]), seed=sum(dims)))
    m = to_np(sim.get_m())
    ref = oracle.heff_terms(problem(*dims, CELL, Ku=500.0), m)["demag"]
    return rel_max(to_np(sim.field("demag")), ref)


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("P", LENGTHS + LONG)
def test_x_lines(P, precision):
    n = (P + 1) // 2
    assert demag_error((n, 3, 1), (P, 0, 0), precision) <= TOL[precision]


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("P", LENGTHS + LONG[:2])  # longer ones exceed the pass's capacity
def test_y_lines_of_thin_grids(P, precision):
    n = (P + 1) // 2
    assert demag_error((3, n, 1), (0, P, 0), precision) <= TOL[precision]


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("P", LENGTHS + LONG[:2])
def test_y_lines_of_thick_grids(P, precision):
    n = (P + 1) // 2
    assert demag_error((2, n, 3), (0, P, 0), precision) <= TOL[precision]


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("P", LENGTHS[1:] + LONG[:2])
def test_z_lines(P, precision):
    n = max(2, (P + 1) // 2)
    assert demag_error((3, 5, n), (0, 0, P), precision) <= TOL[precision]


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("P", [3, 5, 6, 7, 9, 10, 12, 14, 15, 18, 20, 21, 24, 25, 28, 30, 35])
def test_z_lines_in_registers(P, precision):
    # lines of one thread up to 30 points (35: the pass that exchanges through LDS), on
    # planes too large for the fused y-z pass
    n = (P + 1) // 2
    assert demag_error((2, 700 // P + 2, n), (0, 0, P), precision, generic=False) <= TOL[precision]


@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_batch_of_every_length_and_thickness(precision):
    # one handle over grids of 1 to 4 planes whose default padding takes one to four
    # stages along x and y; each grid's field against the direct sum
    grids = [(1, 1, 1), (2, 3, 1), (5, 8, 2), (25, 7, 1), (7, 32, 2), (43, 10, 1), (10, 61, 2), (92, 5, 1),
             (5, 122, 2), (5, 125, 2), (6, 9, 3), (30, 11, 4), (128, 3, 1), (3, 128, 2)]
    hext = np.zeros((len(grids), 3))
    b = mmag.BatchSim(grids, CELL, Ku=500.0, hext=hext, precision=precision)
    assert b.info()["size_classes"] == 0
    b.set_m([random_unit_m((3, g[2], g[1], g[0]), seed=i) for i, g in enumerate(grids)])
    ms, hs = b.get_m(), b.field("demag")
    for g, m, h in zip(grids, ms, hs):
        ref = oracle.heff_terms(problem(*g, CELL, Ku=500.0), to_np(m))["demag"]
        assert rel_max(to_np(h), ref) <= TOL[precision], g
