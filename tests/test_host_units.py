"""Pieces of the library's code that can run on the host, compiled for the host and run there (no GPU)."""
import os
import subprocess

import pytest

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "host")


@pytest.fixture
def run_host(tmp_path):
    def run(name, language=("-x", "hip", "--offload-host-only")):
        exe = str(tmp_path / name)
        subprocess.run(["hipcc", *language, "-O1", "-std=c++17", os.path.join(HERE, name + ".cpp"), "-o", exe], check=True, timeout=300)
        r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
        return r.returncode, r.stdout.strip()
    return run


def test_raw_weight_loads_stay_inside_the_tensor(run_host):
    """1 to 70 channels against weights that end at a page without access: a load past them ends the program."""
    assert run_host("raw_weights") == (0, "ok")


def test_plan_table_keeps_as_many_problems_as_it_holds(run_host):
    """Plans are made once per problem while no more problems take turns than the table has places."""
    assert run_host("plan_table") == (0, "ok")


def test_window_fills_stay_inside_tensor_and_window(run_host):
    """6000 random layers' input ranges, from NCHW and NHWC tensors that touch a page without access on either side."""
    assert run_host("window_fill", ("-x", "c++", "-D__HIP_PLATFORM_AMD__=1", "-I/opt/rocm/include")) == (0, "ok")
