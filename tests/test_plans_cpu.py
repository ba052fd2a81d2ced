"""Which grids do several updates per launch: the grids of the bitwise tests
have to be among them, or those would compare single updates with themselves.
The plan is asked of the built library; no GPU is needed.
"""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from oracle import CLOSED, INFLOW_OUTFLOW, PERIODIC
from paper_2607_20650_amd import lbm
from tests.test_gpu_fused import STRIPS_16_BIT

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    if not os.path.exists(lbm.LIB_PATH):
        pytest.skip("library not built")
    lbm.load_library()
    so = str(tmp_path_factory.mktemp("plan") / "plan.so")
    model = os.path.join(HERE, "host_model")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", model,
                    "-I", os.path.join(ROOT, "paper_2607_20650_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
                    os.path.join(model, "plan.cpp"), lbm.LIB_PATH, "-o", so], check=True)
    return ctypes.CDLL(so)


@pytest.fixture(scope="module")
def plan_of(plans):
    def ask(nx, ny, scheme, layout, precision):
        grid = lbm.Grid(nx, ny, lbm.SCHEMES[scheme], lbm.LAYOUTS[layout], lbm.PRECISIONS[precision], 0, 0)
        bc = lbm.BC(CLOSED, CLOSED, (ctypes.c_double * 2)(), (ctypes.c_double * 2)(), 1.0,
                    (ctypes.c_double * 2)(), 0)
        flags = np.zeros((ny, nx), np.uint8)
        out = (ctypes.c_int32 * 4)()
        assert plans.plan_of(ctypes.byref(grid), ctypes.byref(bc), flags.ctypes.data_as(ctypes.c_void_p), out) == 0
        return dict(kk=out[0], tile=out[1], rows=out[2], own=out[3])

    return ask


@pytest.mark.parametrize("nx,ny,precision,schemes,layouts", STRIPS_16_BIT)
def test_16_bit_grids_run_in_strips(plan_of, nx, ny, precision, schemes, layouts):
    for scheme in schemes:
        for layout in layouts:
            q = plan_of(nx, ny, scheme, layout, precision)
            assert q["kk"] > 1 and not q["tile"], (scheme, layout, q)


@pytest.mark.parametrize("nx,ny,several", [(1000, 601, True), (1300, 1300, False), (2048, 1024, False), (4096, 1024, True)])
def test_fp16s_sr_pull_keeps_single_updates_where_they_are_faster(plan_of, nx, ny, several):
    assert (plan_of(nx, ny, "NPTL", "stream", "fp16sr")["kk"] > 1) == several


@pytest.mark.parametrize("nx,ny,scheme,precision,several", [
    (600000, 1, "NPTL", "fp32", False), (100000, 8, "NPTL", "fp16s", False), (20000, 3, "NPTL", "fp32", True),
    (100000, 8, "AA", "fp16s", True), (100000, 6, "AA", "fp16csr", False), (300000, 2, "NPOL", "fp32", True),
    (300000, 2, "NSOL", "fp16s", False), (1, 100000, "AA", "fp16csr", False), (1, 100000, "AA", "fp32", True),
    (40000, 12, "NPTL", "fp32", True)])
def test_long_grids_of_few_rows(plan_of, nx, ny, scheme, precision, several):
    assert (plan_of(nx, ny, scheme, "stream", precision)["kk"] > 1) == several


@pytest.mark.parametrize("scheme,layout", [("NPTL", "stream"), ("NPTL", "blocked"), ("AA", "stream")])
@pytest.mark.parametrize("nx,ny,nz,axis,several", [
    (201, 97, 85, PERIODIC, True), (201, 97, 85, INFLOW_OUTFLOW, True), (128, 96, 96, INFLOW_OUTFLOW, False),
    (900, 600, 3, PERIODIC, True), (900, 900, 2, PERIODIC, False), (500, 8, 420, INFLOW_OUTFLOW, True),
    (700, 4, 600, INFLOW_OUTFLOW, False), (24, 300, 250, PERIODIC, True), (128, 128, 128, PERIODIC, None),
    (64, 256, 256, PERIODIC, False), (128, 128, 128, INFLOW_OUTFLOW, True),
    (256, 256, 256, PERIODIC, True)])
def test_two_d3q19_updates_per_launch_where_they_are_faster(plans, nx, ny, nz, axis, several, scheme, layout):
    if several is None:
        several = (scheme, layout) == ("NPTL", "stream")
    i64 = ctypes.c_int64
    assert plans.serves3_of(i64(16), i64(320), i64(320), axis, lbm.SCHEMES[scheme], lbm.LAYOUTS[layout]) == (layout == "blocked")
    assert plans.serves3_of(i64(nx), i64(ny), i64(nz), axis, lbm.SCHEMES[scheme], lbm.LAYOUTS[layout]) == several
