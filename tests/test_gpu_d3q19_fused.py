"""Two D3Q19 updates per launch against single updates, bitwise.

``step(1)`` calls launch the scheme's own kernel; one ``step(n)`` runs two
updates per launch where it can.  Both do the same operations per node in the
same order, so every population must be equal bit for bit, on grids that end
inside a tile or a chunk of planes, on every boundary kind.
"""
import numpy as np
import pytest

from oracle import d3q19 as o3
from paper_2607_20650_amd import workloads as W
from tests.helpers import ALL_PRECISIONS

pytestmark = pytest.mark.gpu

P, C, IO = o3.PERIODIC, o3.CLOSED, o3.INFLOW_OUTFLOW
AXES = [(C, C, C), (IO, C, P), (IO, P, C), (P, C, P), (P, P, P)]


def _compare(nx, ny, nz, precision, all_axes, variants):
    from paper_2607_20650_amd.lbm import Simulation3
    flags = W.random_flags3(nx, ny, nz, 0.1, nx + ny)
    st = W.random_state3(nx, ny, nz, 0.02, seed=5, dtype=np.float32)
    for k, axes in enumerate(all_axes):
        if axes[0] == IO and nx < 2:
            continue
        for scheme, layout in variants(k):
            out = []
            for calls in ([1] * 7, [1, 2, 4]):
                with Simulation3(flags, 0.8, *axes, u_in=(0.05, 0.01, -0.01), g=(1e-4, 2e-4, -1e-4),
                                 u0=(0.02, 0.0, 0.01), scheme=scheme, layout=layout, precision=precision) as sim:
                    for n in calls:
                        sim.step(n)
                    sim.set_state(st)
                    for n in calls:
                        sim.step(n)
                    out.append(sim.populations())
            a, b = out
            assert np.array_equal(a, b, equal_nan=True), (axes, scheme, layout, np.argwhere(a != b)[:3])


# from 1.5 million nodes on
@pytest.mark.parametrize("nx,ny,nz", [(70, 67, 330), (5, 560, 560), (2, 900, 900), (1300, 1200, 1), (130, 125, 95),
                                      (900, 900, 2), (1, 1250, 1250), (60, 73, 345)])
def test_two_updates_per_launch_bitwise(nx, ny, nz):
    _compare(nx, ny, nz, "fp32", AXES,
             lambda k: [("NPTL", "stream"), ("NPTL", "blocked"), ("AA", "blocked" if k % 2 else "stream")])


# the fewest rows, planes and columns of a row that do two updates per launch
@pytest.mark.parametrize("nx,ny,nz", [(700, 6, 360), (811, 630, 3), (24, 250, 251), (16, 320, 300)])
def test_two_updates_per_launch_bitwise_thin(nx, ny, nz):
    _compare(nx, ny, nz, "fp32", [AXES[1], AXES[4]],
             lambda k: [("NPTL", "blocked"), ("AA", "blocked")] + ([("NPTL", "stream"), ("AA", "stream")] if nx > 23 else []))


# from 4 million nodes on, x axis not periodic
@pytest.mark.parametrize("precision", [p for p in ALL_PRECISIONS if p != "fp32"])
def test_two_updates_per_launch_bitwise_16_bit(precision):
    _compare(131, 126, 250, precision, AXES[:2],
             lambda k: [("NPTL", "blocked" if k else "stream"), ("AA", "stream" if k else "blocked")])


@pytest.mark.parametrize("scheme", ["NPTL", "AA"])
def test_captured_steps_replay_3d(scheme):
    """As for the 2-D schemes: a captured even number of updates can be
    replayed between eager ones."""
    import torch
    from paper_2607_20650_amd.lbm import Simulation3
    flags = W.random_flags3(130, 100, 120, 0.1, 4)
    kw = dict(u_in=(0.05, 0.01, 0.0), u0=(0.02, 0.0, 0.0), scheme=scheme)
    with Simulation3(flags, 0.8, IO, C, C, **kw) as sim, Simulation3(flags, 0.8, IO, C, C, **kw) as ref:
        sim.step(6)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=sim.stream):
            sim.step(2)
        done = 6
        for _ in range(3):
            with torch.cuda.stream(sim.stream):
                g.replay()
            torch.cuda.synchronize()
            sim.step(4)
            for _ in range(done + 6):
                ref.step(1)
            done = 0
            assert np.array_equal(sim.populations(), ref.populations()), scheme
