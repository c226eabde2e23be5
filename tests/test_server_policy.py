"""The request server's memory policy, on the host: csrc/slg_server.cpp
compiled with stand-ins for the queries' device work (server_policy.cpp)."""
import os
import shutil
import subprocess

import pytest

import paper_2201_11326_amd as slg
from paper_2201_11326_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
CXX = shutil.which("g++") or shutil.which("c++")
ROCM = "/opt/rocm/include"


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not CXX or not os.path.exists(os.path.join(ROCM, "hip", "hip_runtime.h")):
        pytest.skip("no host C++ compiler or no HIP headers")
    exe = str(tmp_path_factory.mktemp("server") / "policy")
    subprocess.run([CXX, "-std=c++17", "-O1", "-w", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I", ROCM,
                    "-I", build.INCLUDE, "-I", build.CSRC, os.path.join(HERE, "server_policy.cpp"), "-o", exe],
                   check=True)

    def run(scenario):
        out = subprocess.run([exe, scenario], capture_output=True, text=True, timeout=60)
        assert out.returncode == 0, (out.returncode, out.stdout, out.stderr)
        *queries, used = out.stdout.splitlines()
        assert used == "used 0"
        assert queries[0] == f"status {slg.SLG_OK} attempts 1 message -"
        return queries[1:]
    return run


def test_a_query_waits_for_its_output(program):
    """With the stores that it could do without, a query waits for room for
    its output where one without such stores does."""
    assert program("output_waits") == [f"status {slg.SLG_OK} attempts 1 message -"]


@pytest.mark.parametrize("scenario", ["stores_refused", "output_fits_without", "output_never_fits_beside"])
def test_a_query_runs_again_without_its_stores(program, scenario):
    """Its stores never make it wait: not for themselves, nor for an output
    that has room without them, now or at all."""
    assert program(scenario) == [f"status {slg.SLG_OK} attempts 2 message -"]


def test_an_output_beyond_the_budget_is_refused(program):
    assert program("output_never_fits") == [f"status {slg.SLG_ERR_OUT_OF_MEMORY} attempts 2 message out of memory"]


@pytest.mark.parametrize("scenario", ["shutdown_after_refusal", "shutdown_after_yield"])
def test_a_query_sent_back_as_the_server_stops_is_cancelled(program, scenario):
    """It would have run again: it has not failed."""
    for line in program(scenario):
        assert line.startswith(f"status {slg.SLG_ERR_CANCELLED} ") and line.endswith("message server shut down")
