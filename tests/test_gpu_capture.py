"""Captured calls replayed between eager ones.

A call captured into a HIP graph holds the addresses it was captured with.
Whatever eager updates run in between (several per launch or not), a replayed
readout has to report the current state and a replayed load has to replace it,
as long as the number of updates since the capture is even.  The reference is
a simulation of single updates (``bundle=0``; in 3-D ``step(1)`` calls), bit
for bit.
"""
import ctypes

import numpy as np
import pytest

from oracle import CLOSED, INFLOW_OUTFLOW
from oracle import d3q19 as o3
from paper_2607_20650_amd import workloads as W
from tests.helpers import ALL_SCHEMES

pytestmark = pytest.mark.gpu

NX, NY = 200, 101
FLOW = dict(u_in=(0.05, 0.01), u0=(0.02, 0.0))


def _pair(scheme):
    from paper_2607_20650_amd.lbm import Simulation
    flags = W.random_flags(NX, NY, 0.1, 4)
    a = Simulation(flags, 0.8, INFLOW_OUTFLOW, CLOSED, scheme=scheme, **FLOW)
    b = Simulation(flags, 0.8, INFLOW_OUTFLOW, CLOSED, scheme=scheme, bundle=0, **FLOW)
    st = W.random_state(NX, NY, 0.02, 3, dtype=np.float32)
    for s in (a, b):
        s.set_state(st)
        s.step(36)
    return a, b


def _ptr(t):
    return ctypes.c_void_p(t.data_ptr())


def _capture(sim, call):
    import torch
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=sim.stream):
        call()
    return g


def _replay(sim, g):
    import torch
    with torch.cuda.stream(sim.stream):
        g.replay()
    torch.cuda.synchronize()


@pytest.mark.parametrize("scheme", ALL_SCHEMES)
def test_captured_readouts_report_the_current_state(scheme):
    import torch
    sim, ref = _pair(scheme)
    f = torch.empty((9, NY, NX), dtype=torch.float32, device="cuda")
    m = torch.empty((3, NY, NX), dtype=torch.float32, device="cuda")
    d = torch.empty(4, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    lib, ctx = sim._lib, sim._ctx

    def readouts():
        sim._check(lib.lbm_get_populations(ctx, _ptr(f), 1))
        sim._check(lib.lbm_macros(ctx, _ptr(m), _ptr(m[1:]), 1))
        sim._check(lib.lbm_diag_noalloc(ctx, None, 0, _ptr(d)))

    g = _capture(sim, readouts)
    for n in (2, 8, 12, 34, 100):  # odd and even numbers of launches
        sim.step(n)
        ref.step(n)
        _replay(sim, g)
        rho, u = ref.macros()
        assert np.array_equal(f.cpu().numpy(), ref.populations()), (scheme, n)
        assert np.array_equal(m.cpu().numpy(), np.concatenate([rho[None], u])), (scheme, n)
        assert d.cpu().numpy().tolist()[:3] == ref.diag()[1][:3], (scheme, n)
        assert np.array_equal(sim.populations(), ref.populations()), (scheme, n)


@pytest.mark.parametrize("scheme", ALL_SCHEMES)
def test_captured_state_load_replaces_the_current_state(scheme):
    import torch
    sim, ref = _pair(scheme)
    st = W.random_state(NX, NY, 0.02, 11, dtype=np.float32)
    dev = torch.from_numpy(st).cuda()
    torch.cuda.synchronize()
    g = _capture(sim, lambda: sim._check(sim._lib.lbm_set_state(sim._ctx, _ptr(dev), 1)))
    for n in (2, 8, 12, 34):
        sim.step(n)
        ref.step(n)
        assert np.array_equal(sim.populations(), ref.populations()), (scheme, n)
        _replay(sim, g)
        ref.set_state(st)
        assert np.array_equal(sim.populations(), ref.populations()), (scheme, n)
        sim.step(6)
        ref.step(6)
        assert np.array_equal(sim.populations(), ref.populations()), (scheme, n)


@pytest.mark.parametrize("scheme", ALL_SCHEMES)
def test_eager_steps_between_capture_and_first_replay(scheme):
    sim, ref = _pair(scheme)
    g = _capture(sim, lambda: sim.step(2))
    for s in (sim, ref):
        s.step(2)
    assert np.array_equal(sim.populations(), ref.populations()), scheme
    for n in (32, 2, 40):
        _replay(sim, g)
        sim.step(n)
        ref.step(2 + n)
        assert np.array_equal(sim.populations(), ref.populations()), (scheme, n)


@pytest.mark.parametrize("scheme", ["NPTL", "AA"])
def test_captured_readouts_and_load_3d(scheme):
    import torch
    from paper_2607_20650_amd.lbm import Simulation3
    nx, ny, nz = 130, 100, 120
    flags = W.random_flags3(nx, ny, nz, 0.1, 4)
    st = W.random_state3(nx, ny, nz, 0.02, seed=5, dtype=np.float32)
    kw = dict(u_in=(0.05, 0.01, 0.0), u0=(0.02, 0.0, 0.0), scheme=scheme)
    axes = (o3.INFLOW_OUTFLOW, o3.CLOSED, o3.CLOSED)
    with Simulation3(flags, 0.8, *axes, **kw) as sim, Simulation3(flags, 0.8, *axes, **kw) as ref:
        m = torch.empty((4, nz, ny, nx), dtype=torch.float32, device="cuda")
        dev = torch.from_numpy(st).cuda()
        torch.cuda.synchronize()
        lib, ctx = sim._lib, sim._ctx

        def ref_step(n):
            for _ in range(n):
                ref.step(1)

        def same(what):
            rho, u = ref.macros()
            _replay(sim, read)
            assert np.array_equal(m.cpu().numpy(), np.concatenate([rho[None], u])), (scheme, what)
            assert np.array_equal(sim.populations(), ref.populations()), (scheme, what)

        sim.step(6)
        ref_step(6)
        read = _capture(sim, lambda: sim._check(lib.lbm3_macros(ctx, _ptr(m), _ptr(m[1:]), 1)))
        load = _capture(sim, lambda: sim._check(lib.lbm3_set_state(ctx, _ptr(dev), 1)))
        for n in (2, 6, 4):
            sim.step(n)
            ref_step(n)
            same(n)
            _replay(sim, load)
            ref.set_state(st)
            same("load")
