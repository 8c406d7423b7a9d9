"""What the library's host side allocates, clears and launches, on a stand-in
of the HIP runtime that runs no kernels (tests/fake_hip): the product library
itself, no GPU."""
import os
import subprocess
import sys

import pytest

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "fake_hip")


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    d = tmp_path_factory.mktemp("fake_hip")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-Wl,-soname,libamdhip64.so.7", "-o", str(d / "libamdhip64.so.7"), os.path.join(HERE, "fake_hip.cpp")],
                   check=True)
    return d


def scenario(runtime, name):
    r = subprocess.run([sys.executable, os.path.join(HERE, "host.py"), name], capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, LD_LIBRARY_PATH=str(runtime)))
    assert r.returncode == 0 and r.stdout.strip().endswith("done"), r.stdout + r.stderr


def test_every_loss_starts_from_cleared_sums(runtime):
    scenario(runtime, "loss_sums")


def test_height_range_needs_no_count_between_workgroups(runtime):
    scenario(runtime, "height_range")


def test_calls_stay_on_their_contexts_device(runtime):
    scenario(runtime, "devices")


def test_reported_bytes_are_the_bytes_held(runtime):
    scenario(runtime, "scene_bytes")


def test_batch_cells_leave_room_and_keep_under_the_cap(runtime):
    scenario(runtime, "batch_cells")
