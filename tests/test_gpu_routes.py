"""Which launches a handle's calls run (mm_get_routes), on both sides of each line of the
dispatch: the plane pass, the fused y-z pass, the fused stage in both forms, the one-launch steps
and the long z lines.  The tests that compare a pass with another or with the oracle rely on it."""
import pytest

mmag = pytest.importorskip("paper_1501_07293_amd")
pytestmark = pytest.mark.gpu

Y, SEP, TWO, PLANE, YZ, WG = range(6)
BOTH = ("f32", "f64")


def routes(dims, precision, **kw):
    sim = mmag.Sim(*dims, 4e-9, precision=precision, **kw)
    r = sim.routes()
    sim.close()
    return r


# 3 nz Py entries a plane: under 3072 up to 8 points along z; up to 2048 from 9 to 12 in FP32; and
# 2^20 (FP64) or 2^21 entries of all bins.  Fused y-z pass: 3 Py Pz up to 4096, or with
# size-specialised passes 2048 (FP64 1024)
MID = [((4, 168, 3), BOTH, PLANE), ((4, 171, 3), BOTH, SEP), ((4, 56, 6), ("f32",), PLANE), ((4, 57, 6), ("f32",), SEP),
       ((4, 56, 6), ("f64",), YZ), ((4, 57, 6), ("f64",), SEP), ((500, 100, 3), ("f64",), PLANE),
       ((1000, 64, 4), ("f64",), SEP), ((1000, 64, 4), ("f32",), PLANE), ((256, 64, 4), BOTH, PLANE),
       ((8, 8, 8), BOTH, YZ), ((8, 16, 8), ("f32",), YZ), ((8, 16, 8), ("f64",), SEP), ((64, 48, 5), ("f64",), YZ),
       ((7, 9, 6), ("f64",), YZ), ((7, 9, 6), ("f32",), PLANE), ((33, 47, 2), BOTH, TWO), ((33, 47, 1), BOTH, Y),
       ((301, 190, 6), BOTH, SEP), ((64, 64, 64), BOTH, SEP)]


@pytest.mark.parametrize("dims,precision,mid", [(d, p, m) for d, ps, m in MID for p in ps])
def test_between_the_x_passes(dims, precision, mid):
    r = routes(dims, precision)
    assert r["mid"] == mid and r["launches"] == (5 if mid == SEP else 3)


def test_asked_for():
    assert routes((300, 8, 6), "f32")["mid"] == PLANE
    assert routes((300, 8, 6), "f32", fused_yz=True) | {"mid": YZ, "launches": 3} == routes((300, 8, 6), "f32", fused_yz=True)
    r = routes((32, 8, 1), "f32", one_wg=True)
    assert (r["mid"], r["launches"], r["stage"], r["one_launch_rk4"]) == (WG, 1, 0, 0)
    for kw in (dict(split_stage=True), dict(generic_fft=True), dict(periodic=(True, False, False)), dict(demag=False)):
        r = routes((32, 8, 1), "f32", **kw)
        assert (r["stage"], r["one_launch_rk4"]) == (0, 0), kw


# size-specialised x lengths up to 2^20 cells, any other of up to 512 points up to 2^17 cells
@pytest.mark.parametrize("precision", BOTH)
@pytest.mark.parametrize("dims,stage", [((128, 128, 1), 1), ((512, 512, 4), 1), ((512, 512, 5), 0), ((30, 30, 1), 2),
                                        ((250, 120, 4), 2), ((250, 524, 1), 2), ((250, 525, 1), 0), ((300, 100, 1), 0),
                                        ((166, 42, 1), 2)])
def test_stage(dims, stage, precision):
    assert routes(dims, precision)["stage"] == stage


# hx Py up to 1024 entries (FP64 256), z not padded
@pytest.mark.parametrize("dims,precision,pz,one", [((27, 18, 1), "f32", 0, 1), ((22, 23, 1), "f32", 0, 0),
                                                   ((8, 8, 1), "f64", 0, 1), ((32, 8, 1), "f64", 0, 0),
                                                   ((32, 8, 1), "f32", 0, 1), ((16, 8, 1), "f32", 4, 0),
                                                   ((8, 8, 1), "f64", 2, 0), ((2, 2, 2), "f32", 0, 0)])
def test_one_launch_steps(dims, precision, pz, one):
    assert routes(dims, precision, pad=(0, 0, pz))["one_launch_rk4"] == one


# power-of-two lines of 128 points or more; the wide form from 2 GiB on (spectrum, then octant)
@pytest.mark.parametrize("dims,precision,pad,form", [((64, 64, 64), "f32", (0, 0, 0), 1), ((8, 8, 8), "f32", (64, 512, 128), 1),
                                                     ((8, 8, 64), "f32", (1024, 2744, 128), 2),
                                                     ((8, 8, 2), "f64", (1024, 1024, 512), 2),
                                                     ((8, 512, 32), "f32", (0, 0, 64), 0), ((8, 8, 8), "f64", (64, 512, 1024), 0)])
def test_long_z(dims, precision, pad, form):
    assert routes(dims, precision, pad=pad)["long_z"] == form
