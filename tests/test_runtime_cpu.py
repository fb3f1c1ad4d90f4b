"""The library's host side on a HIP runtime without a device (fake_hip.cpp):
what is uploaded, kept and refused where calls of the runtime fail."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def fake(qtn, tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("fake") / "fake_hip")
    lib = os.path.join(ROOT, "paper_2204_06045_amd")
    # the program's definitions come before those of the runtime library
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", ROCM + "/include",
                    "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "fake_hip.cpp"), "-o", exe, "-rdynamic", "-L", lib,
                    "-lqtn", "-Wl,-rpath," + lib, "-Wl,-rpath," + ROCM + "/lib",
                    "-Wl,--allow-shlib-undefined"], check=True)
    return exe


def _run(fake, scenario):
    r = subprocess.run([fake, scenario], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


def test_refused_call_leaves_no_descriptors_behind(fake):
    # a schedule's descriptors go up once: a copy that a capture swallowed must
    # not count
    _run(fake, "refused_under_capture")


def test_failed_descriptor_allocation_is_tried_once(fake):
    _run(fake, "no_memory_for_descriptors")


def test_descriptors_of_many_batches_are_bounded(fake):
    _run(fake, "descriptors_of_many_batches")


def test_autotuner_times_the_mappings_it_picks(fake):
    _run(fake, "autotuned_small_groups")


def test_autotuner_keeps_step_launches(fake):
    _run(fake, "autotuned_steps")
