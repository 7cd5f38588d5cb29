"""The fused stage pass and its adjoint at x lengths without a size-specialised pass, and
the fused y-z pass on small planes, against the separate passes (MM_SPLIT_STAGE with the
runtime-radix family, which on these grids takes y forward, z k-space and y inverse apart or
in one by the plane's size) and against the oracle."""
import numpy as np
import pytest

import oracle
from synthetic import mT_to_Apm, random_unit_m
from tests.gpu_util import rel_max, to_np

pytestmark = pytest.mark.gpu

mmag = pytest.importorskip("paper_1501_07293_amd")


def make(dims, precision, **kw):
    s = mmag.Sim(*dims, 4e-9, Ku=2e3, alpha=0.3, precision=precision, **kw)
    s.set_hext(mT_to_Apm([5.0, -3.0, 2.0]))
    return s


# one, two and four row pairs a work-group (under 1024, 2048 rows and more); one and two
# cells a thread; rows that leave a block ragged; odd and even lengths of one to four stages
# up to 500 points; one column; planes at the fused y-z pass's limit on both sides
GRIDS = [(30, 30, 1), (7, 5, 1), (1, 9, 1), (45, 61, 1), (166, 42, 1), (250, 33, 1), (100, 100, 1), (18, 1023, 1),
         (21, 1025, 1), (5, 1030, 2), (50, 50, 2), (60, 40, 3), (27, 35, 7), (98, 25, 10), (12, 12, 12), (33, 682, 2)]


@pytest.mark.parametrize("dims", GRIDS)
@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_matches_separate_passes(dims, precision):
    one, apart = make(dims, precision), make(dims, precision, split_stage=True)
    m0 = random_unit_m((3, dims[2], dims[1], dims[0]), seed=sum(dims))
    for s in (one, apart):
        s.set_m(m0)
        s.step(9, 1e-13)
        s.step_euler(3, 1e-14)
    # rounding of two orders of the same operations over 39 field evaluations
    assert np.abs(to_np(one.get_m()) - to_np(apart.get_m())).max() <= (1e-13 if precision == "f64" else 2e-6)


@pytest.mark.parametrize("dims", [(30, 14, 1), (15, 9, 3), (10, 7, 2)])
@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_trajectory_and_adjoint_match_oracle(dims, precision):
    import torch
    g = np.random.default_rng(7)
    nx, ny, nz = dims
    ku = 500.0 + 50.0 * g.standard_normal((nz, ny, nx))
    hext = mT_to_Apm([6.0, -2.0, 4.0])
    pb = oracle.Problem(nx, ny, nz, 5e-9, Ku=0.0, alpha=0.1, ku_map=ku, hext=tuple(hext))
    sim = mmag.Sim(nx, ny, nz, 5e-9, Ms=pb.Ms, A=pb.A, Ku=0.0, alpha=pb.alpha, gamma=pb.gamma, precision=precision)
    sim.set_hext(hext)
    sim.set_ku_map(ku)
    sim.set_m(random_unit_m(pb.shape, 4))
    m_used = to_np(sim.get_m())
    w = g.standard_normal(pb.shape)
    dt, nsteps, ck = 1e-13, 11, 4
    ckpt = sim.rollout_ckpt(nsteps, dt, ck)
    assert np.abs(to_np(sim.get_m()) - oracle.rk4(pb, m_used, dt, nsteps)).max() <= (1e-11 if precision == "f64" else 1e-5)
    lam = torch.tensor(w, dtype=sim.dtype, device=sim.device)
    dku, dm0 = sim.backward(nsteps, dt, ck, ckpt, lam)
    ref_ku, ref_m0 = oracle.rk4_adjoint(pb, m_used, dt, nsteps, w)
    tol = 1e-9 if precision == "f64" else 1e-4
    assert rel_max(to_np(dku), ref_ku) <= tol
    assert rel_max(to_np(dm0), ref_m0) <= tol


@pytest.mark.parametrize("dims", [(45, 20, 1), (30, 12, 3)])
@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_graph_replay_equals_plain_launches(dims, precision):
    # several replays with eager work and synchronisation between them
    plain, graph = make(dims, precision), make(dims, precision, graph=True)
    m0 = random_unit_m((3, dims[2], dims[1], dims[0]), seed=5)
    for s in (plain, graph):
        s.set_m(m0)
    for _ in range(3):
        for s in (plain, graph):
            s.step(35, 1e-13)
            s.field("eff")
            s.step_euler(19, 1e-14)
        assert np.array_equal(to_np(plain.get_m()), to_np(graph.get_m()))
