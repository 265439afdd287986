"""The order that compress calls leave between streams, and the shapes of launches, without a GPU: the library's host code is
driven on a double of the HIP runtime (host_order.cpp) that keeps what every launch and copy is ordered behind.
"""
import os
import subprocess

import pytest

from paper_2410_20650_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host_order") / "host_order")
    csrc = os.path.join(ROOT, "paper_2410_20650_amd", "csrc")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-rdynamic", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", csrc,
           "-I", os.path.join(ROOT, "include"), os.path.join(HERE, "host_order.cpp"), build.BUILT_LIB,
           "-Wl,-rpath," + os.path.dirname(build.BUILT_LIB), "-Wl,--allow-shlib-undefined", "-o", exe]
    built = subprocess.run(cmd, capture_output=True, text=True)
    assert built.returncode == 0, built.stderr
    return exe


def run(driver, scenario):
    done = subprocess.run([driver, scenario], capture_output=True, text=True, timeout=120)
    assert done.returncode == 0 and done.stdout.strip().endswith("ok"), done.stdout + done.stderr


@pytest.mark.parametrize("scenario", ["failure", "failure_in_a_tile"])
def test_a_failed_call_is_behind_the_next_one_on_another_stream(driver, scenario):
    run(driver, scenario)


@pytest.mark.parametrize("scenario", ["other_stream", "other_stream_in_tiles", "batch"])
def test_calls_that_read_a_blob_are_behind_the_call_that_fills_it(driver, scenario):
    run(driver, scenario)


@pytest.mark.parametrize("scenario", ["nothing_to_wait_for", "capture"])
def test_no_event_where_there_is_nothing_to_wait_for(driver, scenario):
    run(driver, scenario)


def test_an_old_stamp_is_not_taken_for_this_calls(driver):
    run(driver, "old_stamp")


def test_a_decoders_workgroup_has_as_many_chunks_as_fit(driver):
    run(driver, "chunks_of_a_workgroup")


@pytest.mark.parametrize("scenario", ["form_of_the_walk", "form_of_the_whole_walk", "form_of_the_linear_walk"])
def test_the_form_of_the_walk(driver, scenario):
    run(driver, scenario)


def test_the_columns_of_the_linear_walk_with_and_without_scratch_memory(driver):
    run(driver, "columns_of_the_linear_walk")
