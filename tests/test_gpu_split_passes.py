"""The passes that do several at once against the ones they stand for, each side's route checked:
fused y-z and plane pass against y forward, z k-space and y inverse (split_yz); and the one-launch
steps over more steps than one launch takes against the same run in several calls."""
import numpy as np
import pytest

from synthetic import random_unit_m
from tests.gpu_util import rel_max, to_np

mmag = pytest.importorskip("paper_1501_07293_amd")
pytestmark = pytest.mark.gpu

CELL = 4e-9
# both sides' transforms, lines of up to 2^13 points in all: some 30 eps of the largest entry each
FIELD_TOL = {"f32": 4e-6, "f64": 4e-14}
# 40 evaluations a side, each moving m by under 0.1 of a unit per unit of the field
STEP_TOL = {"f32": 1.6e-5, "f64": 1.6e-13}


def sim(dims, precision, **kw):
    return mmag.Sim(*dims, CELL, Ku=2e3, alpha=0.3, precision=precision, **kw)


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("dims,kw", [((256, 64, 4), {}), ((20, 15, 3), {}), ((64, 48, 5), {}), ((100, 30, 2), {}),
                                     ((7, 9, 6), {}), ((8, 8, 8), {}), ((12, 12, 12), {}),
                                     ((27, 35, 7), dict(generic_fft=True)), ((20, 12, 6), dict(periodic=(True, True, True)))])
def test_one_pass_for_three(dims, kw, precision):
    apart = sim(dims, precision, split_yz=True, **kw)
    assert apart.routes()["mid"] == mmag.MID_SEPARATE and apart.routes()["launches"] == 5
    m0 = random_unit_m((3, dims[2], dims[1], dims[0]), seed=sum(dims))
    apart.set_m(m0)
    ref = to_np(apart.field("demag"))
    apart.step(10, 1e-13)
    m = to_np(apart.get_m())
    for one in (sim(dims, precision, **kw), sim(dims, precision, fused_yz=True, **kw)):
        assert one.routes()["mid"] in (mmag.MID_PLANE, mmag.MID_FUSED_YZ) and one.routes()["launches"] == 3
        one.set_m(m0)
        assert rel_max(to_np(one.field("demag")), ref) <= FIELD_TOL[precision]
        one.step(10, 1e-13)
        assert np.abs(to_np(one.get_m()) - m).max() <= STEP_TOL[precision]


def test_split_yz_takes_precedence():
    assert sim((64, 48, 5), "f32", fused_yz=True, split_yz=True).routes()["mid"] == mmag.MID_SEPARATE
    assert sim((33, 47, 2), "f32", split_yz=True).routes()["mid"] == mmag.MID_TWO_PLANE


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_one_launch_steps_past_one_launch(precision, graph):
    # 4096 steps a launch: the state leaves the work-group unrounded, so any split of a run into
    # calls gives the same bits
    out = []
    for calls in ((4096 + 4096 + 5,), (4096, 1, 4096, 4), (1000, 7197)):
        s = sim((8, 8, 1), precision, graph=graph)
        assert s.routes()["one_launch_rk4"] == 1
        s.set_m(random_unit_m((3, 1, 8, 8), seed=2))
        s.set_hext((1e4, -2e4, 3e4))
        for n in calls:
            s.step(n, 1e-13)
        out.append(to_np(s.get_m()))
    assert np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2])
    assert np.isfinite(out[0]).all() and np.abs(np.linalg.norm(out[0], axis=0) - 1).max() < 1e-5
