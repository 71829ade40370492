"""State that the host side keeps between calls, on a stand-in device (see
host_state.cpp): a workspace whose first clearing failed or was captured, a
sequence of launches that stops half way, allocations that fail,
growths and conversions whose lists prove too short.

Needs a host compiler and the HIP headers, no GPU.
"""
import os
import shutil
import subprocess

import pytest

from conftest import ROOT

ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
SCENARIOS = ["first_call_captured", "clearing_fails", "sequence_stops", "graph_calls",
             "allocation_fails", "growth_list_fails", "refused_allocation_is_reported_once",
             "lists_too_short"]


@pytest.fixture(scope="module")
def stand_in(tmp_path_factory):
    if not shutil.which("g++") or not os.path.isdir(os.path.join(ROCM, "include", "hip")):
        pytest.skip("no host compiler or HIP headers")
    out = str(tmp_path_factory.mktemp("host_state") / "host_state")
    cmd = ["g++", "-std=c++17", "-O1", "-Wno-unused-result", "-D__HIP_PLATFORM_AMD__",
           "-I", os.path.join(ROCM, "include"), "-x", "c++",
           os.path.join(ROOT, "paper_2106_08150_amd", "csrc", "mc_api.hip"),
           os.path.join(ROOT, "tests", "host_state.cpp"), "-o", out, "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    return out


@pytest.mark.parametrize("name", SCENARIOS)
def test_host_state(stand_in, name):
    r = subprocess.run([stand_in, name], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
