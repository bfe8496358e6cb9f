"""Index arithmetic of the row kernels that read column codes, on the host: every
load in range and every row taken once, over all remainders of a block of rows."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("coded_rows") / "coded_rows")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_2007_00056_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "coded_rows.cpp"), "-o", exe], check=True)
    return lambda *args: subprocess.run([exe, *map(str, args)], capture_output=True, text=True)


@pytest.mark.parametrize("first,last", [(1, 700), (4000, 4600)])
def test_every_load_in_range(walk, first, last):
    r = walk(first, last)
    assert r.returncode == 0, r.stdout


def test_waves_past_the_matrix_have_to_be_left_out(walk):
    """The walk sees the reads that a wave past the last row would make with the last slice's distances."""
    r = walk(4097, 4400, "all-waves")
    assert r.returncode > 0, r.stdout
