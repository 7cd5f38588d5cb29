"""Host checks of mm_get_routes and of what bench.py makes of it (no GPU): the binding's struct
and constants against the header, the bytes and kernel names of routed plans."""
import ctypes
import os
import re
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402
import paper_1501_07293_amd as mm  # noqa: E402

HEADER = open(os.path.join(ROOT, "include", "mmag.h")).read()


def test_struct_and_constants_match_the_header():
    body = HEADER[:HEADER.index("} mm_route_info;")]
    body = re.sub(r"/\*.*?\*/", "", body[body.rindex("typedef struct {"):], flags=re.S)
    assert re.findall(r"int32_t (\w+);", body) == [n for n, _ in mm.RouteInfo._fields_]
    assert all(t is ctypes.c_int32 for _, t in mm.RouteInfo._fields_)
    consts = dict(re.findall(r"\bMM_((?:MID|STAGE|ZLINE)_\w+) = (\d+)", HEADER))
    assert len(consts) == 12
    for name, value in consts.items():
        assert getattr(mm, name) == int(value), name


def test_null_arguments_are_refused():
    lib = mm.load_library()
    assert lib.mm_get_routes(None, ctypes.byref(mm.RouteInfo())) == -1


PLAN = {"px": 512, "py": 128, "pz": 8, "hx": 257, "passes": 5, "threads": 256, "generic_fft": 0, "x_lines": 8,
        "x_lines_inv": 4, "spectrum_elems": 6 * 5 * 257 * 65, "fused_stage": 1, "stage": 1, "one_launch_rk4": 0,
        "long_z": 0}


@pytest.mark.parametrize("mid,launches,name", [(mm.MID_PLANE, 3, "mm::k_plane"), (mm.MID_FUSED_YZ, 3, "mm::k_ryz"),
                                               (mm.MID_SEPARATE, 5, "mm::k_kspace_z<float, 8>")])
def test_bench_takes_the_passes_that_run(mid, launches, name):
    plan = dict(PLAN, mid=mid, launches=launches)
    assert bench.mm_kernel_symbol("kspace", "f32", plan, (256, 64, 4)) == name
    assert bench.kernel_digest(name)
    b = bench.algorithmic_bytes(plan, 256, 64, 4, 4)
    half, full = 3 * 4 * 64 * 257 * 8, 3 * 4 * 128 * 257 * 8
    kern = PLAN["spectrum_elems"] * 4
    assert b["kspace"] == (2 * half + kern if launches == 3 else 2 * full + kern)
    assert b["y_fwd"] == b["y_inv"] == (0 if launches == 3 else half + full)


def test_bench_names_the_runtime_length_passes():
    plan = dict(PLAN, px=600, py=380, pz=12, stage=2, mid=mm.MID_SEPARATE, launches=5)
    sym = lambda k, **kw: bench.mm_kernel_symbol(k, "f32", dict(plan, **kw), (300, 190, 6))
    names = {k: sym(k) for k in bench.KERNEL_IDS}
    assert names == {"x_fwd": "mm::k_rxfwd", "x_inv": "mm::k_rxinv", "y_fwd": "mm::k_ryline", "y_inv": "mm::k_ryline",
                     "kspace": "mm::k_kspace_z_mixed<float, 12>", "llg": "mm::k_rfused_stage"}
    assert sym("kspace", pz=200) == "mm::k_rkz" and sym("kspace", mid=mm.MID_Y, pz=1, launches=3) == "mm::k_rky"
    assert sym("kspace", pz=256, long_z=2) == "mm::k_kspace_zl_wide<float, 256>"
    assert all(bench.kernel_digest(n) for n in list(names.values()) + ["mm::k_rkz", "mm::k_rky", "mm::kbr_x<"])
