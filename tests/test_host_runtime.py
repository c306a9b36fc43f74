"""The host runtime's loops, group sizes and refusals, without a GPU: bfs_host.cpp
compiled by g++ against a HIP runtime and kernels that only keep count
(tests/host_runtime.cpp)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(f"{ROCM}/include/hip"),
                                reason="needs g++ and the HIP headers")


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "host_runtime")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include", "-w",
                    "-o", exe, os.path.join(HERE, "host_runtime.cpp")], check=True)
    return exe


def run(exe, case):
    r = subprocess.run([exe, case], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


def test_step_loop_ends_for_any_levels_per_sync(runtime):
    run(runtime, "steps")


def test_deep_batches_of_any_size(runtime):
    run(runtime, "deep_groups")


def test_deep_launches_past_the_end(runtime):
    run(runtime, "deep_syncs")


def test_form_of_a_batch_on_thin_graphs(runtime):
    run(runtime, "deep_choice")


def test_network_asked_once_a_decision(runtime):
    run(runtime, "ms_decisions")


def test_form_of_a_push_on_graphs_with_hubs(runtime):
    run(runtime, "sliced_choice")


def test_form_of_a_push_on_even_degrees(runtime):
    run(runtime, "even_choice")


def test_planes_become_levels_where_they_fit(runtime):
    run(runtime, "levels_fit")
