"""Device code built for the CPU with an emulation of one workgroup (simt.hpp), where what is asked is what lanes
that have left a loop do, or inputs that must not reach a GPU."""
import os
import subprocess

import pytest

from paper_2506_16235_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))
CLANG = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(B.HIPCC))), "llvm", "bin", "clang++")


def _run(tmp_path, source):
    if not os.path.exists(CLANG):
        pytest.skip("no clang++")
    exe = str(tmp_path / "driver")
    subprocess.run([CLANG, "-O1", "-std=c++17", "-Wall", "-Wno-unused", "-Wno-unknown-pragmas", "-ffp-contract=off", "-I", B.INCLUDE, "-I", B.CSRC,
                    os.path.join(HERE, source), "-o", exe, "-lm"], check=True, capture_output=True)
    p = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, p.stdout + p.stderr


def test_sampled_counts_are_those_of_a_plain_histogram(tmp_path):
    _run(tmp_path, "sample_driver.cpp")


def test_dense_passes_notice_a_wrong_count_before_they_write(tmp_path):
    _run(tmp_path, "dense_driver.cpp")


def test_first_survivor_of_a_tile_by_a_wavefront(tmp_path):
    _run(tmp_path, "search_driver.cpp")
