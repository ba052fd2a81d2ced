"""Host code of the simulation contexts and the serving engine on a modelled
device.

``csrc/context.hip``, ``csrc/context3.hip`` and ``csrc/server.hip`` hold no
kernels, so they compile with g++ against a model of the HIP runtime
(``host_model/hip/hip_runtime.h``) and of the launches (``host_model/model.cpp``):
device memory has addresses and every lattice holds its update count instead of
populations.  Each scenario checks that the addresses, the order and the
lifetimes the contexts use belong together, also where a GPU could only show a
mistake by a fault.
"""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
MODEL = os.path.join(HERE, "host_model")
CSRC = os.path.join(ROOT, "paper_2607_20650_amd", "csrc")


@pytest.fixture(scope="module")
def scenarios(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host_model") / "scenarios")
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", MODEL, "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                    "-x", "c++", *(os.path.join(CSRC, f) for f in ("context.hip", "context3.hip", "server.hip")),
                    os.path.join(MODEL, "model.cpp"), os.path.join(MODEL, "scenarios.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("name", ["captured_readout", "captured_load", "eager_before_replay", "captured_3d",
                                  "graphs_after_capture", "calls_of_one_update", "given_back", "given_back_to_others",
                                  "given_back_across_threads", "spare_memory_is_bounded", "readout_from_another_device",
                                  "served_single_updates", "served_by_load"])
def test_scenario(scenarios, name):
    r = subprocess.run([scenarios, name], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout[:2000]
