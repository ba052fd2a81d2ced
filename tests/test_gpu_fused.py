"""Several updates per launch against single updates, bitwise.

With ``bundle=0`` every update is a launch of the scheme's own kernel; the
default runs several updates per launch (tiles on small grids, marching strips
on large ones).  Both do the same operations per node in the same order, so
every population must be equal bit for bit, on grids that end inside a tile, a
strip, a block of strips or a chunk of rows, on every boundary kind.
"""
import numpy as np
import pytest

from oracle import CLOSED, INFLOW_OUTFLOW, INFLOW_PRESSURE, NEUMANN_OUTFLOW, PERIODIC
from paper_2607_20650_amd import workloads as W
from tests.helpers import ALL_LAYOUTS, ALL_PRECISIONS

pytestmark = pytest.mark.gpu

AXES = [(PERIODIC, PERIODIC), (CLOSED, CLOSED), (INFLOW_OUTFLOW, CLOSED), (INFLOW_PRESSURE, PERIODIC),
        (CLOSED, PERIODIC), (PERIODIC, CLOSED), (NEUMANN_OUTFLOW, CLOSED)]


def _run(sim_cls, nx, ny, xa, ya, bundle, calls, **kw):
    flags = W.random_flags(nx, ny, 0.1, nx + ny)
    st = W.random_state(nx, ny, 0.02, 3, dtype=np.float32)
    with sim_cls(flags, 0.8, xa, ya, u_in=(0.05, 0.01), g=(1e-4, 2e-4), u0=(0.02, 0.0), bundle=bundle, **kw) as sim:
        sim.set_state(st)
        for n in calls:
            sim.step(n)
        return sim.populations()


def _compare(nx, ny, axes, schemes, layouts, precisions, calls=(4, 7, 1, 19, 3, 2)):
    from paper_2607_20650_amd.lbm import Simulation
    for xa, ya in axes:
        if xa >= INFLOW_OUTFLOW and nx < 2:
            continue
        for scheme in schemes:
            for layout in layouts:
                for prec in precisions:
                    kw = dict(scheme=scheme, layout=layout, precision=prec)
                    a = _run(Simulation, nx, ny, xa, ya, 0, calls, **kw)
                    b = _run(Simulation, nx, ny, xa, ya, 16, calls, **kw)
                    assert np.array_equal(a, b, equal_nan=True), (nx, ny, xa, ya, kw, np.argwhere(a != b)[:3])


@pytest.mark.parametrize("precision", ALL_PRECISIONS)
@pytest.mark.parametrize("nx,ny", [(128, 64), (37, 20), (5, 3), (1, 7), (2, 2), (50, 33), (57, 5), (200, 101)])
def test_small_grids_bitwise(nx, ny, precision):
    _compare(nx, ny, AXES, ["NPTL", "PUSH"], ALL_LAYOUTS, [precision])


@pytest.mark.parametrize("precision", ALL_PRECISIONS)
@pytest.mark.parametrize("nx,ny", [(2311, 701), (193, 8300), (200003, 9), (410001, 4), (13, 125003)])
def test_large_grids_bitwise(nx, ny, precision):
    _compare(nx, ny, AXES[:4], ["NPTL", "PUSH"], ["stream"], [precision], calls=(8, 5, 17))


def test_large_grid_layouts_bitwise():
    _compare(2311, 701, AXES[2:4], ["LPTL", "NPTL", "PUSH"], ["bundle", "collision"], ["fp32", "fp16sr", "fp16c"],
             calls=(8, 5))
    # FP32 from 3 million nodes on: eight updates per launch
    _compare(3011, 1003, AXES[1:4], ["NPTL", "PUSH", "AA", "NSOL"], ["stream"], ["fp32"], calls=(16, 13))


# 16-bit formats on grids of several updates per launch in strips (checked
# without a GPU in test_plans_cpu.py): nx, ny, precision, schemes, layouts.
# FP16C in NPTL and in stream AA and PUSH has them beyond 256 MB of lattices,
# the FP16S-SR pull of NPTL beyond 2.4 million nodes.
STRIPS_16_BIT = [
    (2311, 701, "fp16c", ["PUSH", "AA"], ["bundle", "collision"]),
    (2311, 701, "fp16csr", ["PUSH", "AA", "LPTL"], ["bundle", "collision"]),
    (2311, 701, "fp16sr", ["PUSH", "AA", "LPTL"], ["stream", "collision"]),
    (2311, 701, "fp16c", ["LPTL"], ["stream", "bundle"]),
    (3011, 1003, "fp16sr", ["NPTL"], ["stream", "bundle"]),
    (3011, 2515, "fp16c", ["NPTL", "AA", "PUSH"], ["stream"]),
    (3011, 2515, "fp16csr", ["NPTL", "AA", "PUSH"], ["stream"]),
]


@pytest.mark.parametrize("nx,ny,precision,schemes,layouts", STRIPS_16_BIT)
def test_16_bit_strips_bitwise(nx, ny, precision, schemes, layouts):
    _compare(nx, ny, AXES[2:3], schemes, layouts, [precision], calls=(8, 5))


@pytest.mark.parametrize("precision", ALL_PRECISIONS)
@pytest.mark.parametrize("nx,ny", [(128, 64), (37, 20), (5, 3), (57, 5), (200, 101), (2311, 701), (200003, 9), (13, 125003)])
def test_one_lattice_schemes_bitwise(nx, ny, precision):
    """AA in pairs of updates, NPOL and NSOL without their edge buffers, from
    odd and even update counts, and back to single updates in between."""
    from paper_2607_20650_amd.lbm import Simulation
    small = nx * ny < 100000
    for xa, ya in AXES if small else AXES[1:3]:
        flags = W.random_flags(nx, ny, 0.1, nx + ny)
        st = W.random_state(nx, ny, 0.02, 3, dtype=np.float32)
        for scheme in ["AA", "NPOL", "NSOL"]:
            for layout in ALL_LAYOUTS if small else ["stream"]:
                out = []
                for bundle in (0, 16):
                    kw = dict(scheme=scheme, layout=layout, precision=precision)
                    with Simulation(flags, 0.8, xa, ya, u_in=(0.05, 0.01), g=(1e-4, 2e-4), u0=(0.02, 0.0),
                                    bundle=bundle, **kw) as sim:
                        sim.step(5)
                        sim.step(19)
                        a = sim.populations()
                        sim.set_state(st)
                        sim.step(8)
                        sim._check(sim._lib.lbm_set_bundle(sim._ctx, 0))
                        sim.step(3)
                        sim._check(sim._lib.lbm_set_bundle(sim._ctx, bundle))
                        sim.step(6)
                        out.append((a, sim.populations()))
                for a, b in zip(*out):
                    assert np.array_equal(a, b, equal_nan=True), (nx, ny, xa, ya, kw, np.argwhere(a != b)[:3])


@pytest.mark.parametrize("scheme", ["NPOL", "NSOL"])
@pytest.mark.parametrize("nx,ny,layout,precision", [(3011, 1003, "stream", "fp32"), (700, 501, "collision", "fp16sr"),
                                                    (2311, 701, "bundle", "fp16s"), (3001, 2501, "stream", "fp16c")])
def test_calls_of_one_update_bitwise(nx, ny, layout, precision, scheme):
    """Calls of one update run the scheme's own kernel on these grids (NSOL in
    16 bits beyond 256 MB), between launches of several."""
    _compare(nx, ny, AXES[2:3], [scheme], [layout], [precision], calls=(1, 1, 8, 1, 1, 1, 6, 1))


@pytest.mark.parametrize("scheme", ["NPTL", "PUSH", "AA", "NPOL", "NSOL"])
def test_captured_steps_replay(scheme):
    """A captured call of an even number of updates can be replayed, with eager
    steps and readouts in between: it finds the state where it left it."""
    import torch
    from paper_2607_20650_amd.lbm import Simulation
    flags = W.random_flags(200, 101, 0.1, 4)
    st = W.random_state(200, 101, 0.02, 3, dtype=np.float32)
    kw = dict(u_in=(0.05, 0.01), u0=(0.02, 0.0), scheme=scheme)
    with Simulation(flags, 0.8, INFLOW_OUTFLOW, CLOSED, **kw) as sim, \
            Simulation(flags, 0.8, INFLOW_OUTFLOW, CLOSED, bundle=0, **kw) as ref:
        for s in (sim, ref):
            s.set_state(st)
            s.step(36)  # several updates per launch so far
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=sim.stream):
            sim.step(2)
        for k in range(4):
            with torch.cuda.stream(sim.stream):
                g.replay()
            torch.cuda.synchronize()
            ref.step(2)
            assert np.array_equal(sim.populations(), ref.populations()), (scheme, k)
            sim.step(34)
            ref.step(34)
            assert np.array_equal(sim.populations(), ref.populations()), (scheme, k)


def test_spare_memory_goes_back():
    """A server pool that cannot be had takes the second lattices and link words
    of the simulations with it; they go on in place, bit for bit."""
    from paper_2607_20650_amd.lbm import ENOMEM, LbmError, Server, Simulation, Simulation3
    flags, flags3 = W.random_flags(2311, 701, 0.1, 4), W.random_flags3(130, 125, 95, 0.1, 4)
    kw = dict(u_in=(0.05, 0.01), u0=(0.02, 0.0))
    kw3 = dict(u_in=(0.05, 0.01, 0.0), u0=(0.02, 0.0, 0.0), scheme="AA")
    axes3 = (INFLOW_OUTFLOW, CLOSED, CLOSED)
    refs = [Simulation(flags, 0.8, INFLOW_OUTFLOW, CLOSED, scheme="NPTL", bundle=0, **kw),
            Simulation3(flags3, 0.8, *axes3, **kw3)]
    sims = [Simulation(flags, 0.8, INFLOW_OUTFLOW, CLOSED, scheme=s, **kw) for s in ("AA", "NPOL", "NSOL")]
    sim3 = Simulation3(flags3, 0.8, *axes3, **kw3)
    held = [s.info()["device_bytes"] for s in sims]
    for s in sims + [sim3]:
        s.step(6)  # one launch (two-dimensional): the state is in the second lattice
    with pytest.raises(LbmError) as e:
        Server(1 << 45)
    assert e.value.status == ENOMEM
    for s, before in zip(sims, held):
        assert s.info()["device_bytes"] < before
    for n in (1, 9, 16):
        for s in sims + [sim3]:
            s.step(n)
    refs[0].step(32)
    for _ in range(32):
        refs[1].step(1)
    for s in sims:
        assert np.array_equal(s.populations(), refs[0].populations()), s.scheme
    assert np.array_equal(sim3.populations(), refs[1].populations())
    for s in sims + refs + [sim3]:
        s.close()
