"""The encoder's step that codes nothing, and its limits, without a GPU; and that the tensors of high_states.py are what they
are made for.
"""
import os
import subprocess

import numpy as np
import pytest

import high_states as H
from oracle import oracle as O
from paper_2410_20650_amd import inputs

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_limits_and_the_step_that_codes_nothing(tmp_path):
    exe = str(tmp_path / "encoder_step")
    cmd = ["g++", "-std=c++17", "-O2", "-Wall", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
           "-I", os.path.join(ROOT, "paper_2410_20650_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
           os.path.join(HERE, "encoder_step.cpp"), "-o", exe]
    built = subprocess.run(cmd, capture_output=True, text=True)
    assert built.returncode == 0, built.stderr
    done = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert done.returncode == 0 and done.stdout.strip().endswith("ok"), done.stdout + done.stderr


@pytest.mark.parametrize("end", [7, 127, 2048 + 8])
def test_the_lanes_that_are_made_to_end_high_do(end):
    words = inputs.bits(inputs.gaussian_bf16(3 * 4096 + end, 7000 + end))
    freq = O.blob_info(O.compress(words, 7, threads=4))["freq"]
    got = H.end_on_high_states(words, end, freq, H.Bf16, end)
    container = O.compress(got, 7, threads=4)
    assert H.high_lanes(container, end) == [j for j, _, n in H.tail_lanes(end) if n >= 7]
    assert np.array_equal(O.decompress(container, got.size), got)
