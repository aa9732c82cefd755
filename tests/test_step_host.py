"""CPU tests of the host side of lbm_step_ws and of the rules for passes
(tests/host/step_paths.cpp): the library's own code over a HIP runtime that
records launches instead of running them."""
import os
import subprocess

import pytest

import pass_shapes

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "host", "step_paths.cpp")
LIB_DIR = os.path.join(ROOT, "paper_1611_03329_amd")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("host") / "step_paths")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-O1", "-rdynamic", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"),
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(LIB_DIR, "csrc"), SRC, "-o", out, os.path.join(LIB_DIR, "liblbm.so"),
                    "-Wl,-rpath," + LIB_DIR, "-Wl,-rpath-link," + os.path.join(rocm, "lib")], check=True)
    return out


@pytest.mark.parametrize("scenario", ["capture", "offered", "failed", "marching", "step_order", "query_order"])
def test_host_side_of_passes(program, scenario):
    r = subprocess.run([program, scenario], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.parametrize("table", ["FLOW", "MELT", "MARCH"])
def test_the_boxes_of_the_gpu_tests_reach_their_kernels(program, table):
    for name, row in getattr(pass_shapes, table).items():
        shape, kernels = row[0], row[-1]
        for prec, want in kernels.items():
            args = ["kernel", table, str(["fp64", "fp32", "fp16"].index(prec)), *map(str, shape)]
            got = subprocess.run([program, *args], capture_output=True, text=True, timeout=60, check=True).stdout
            assert int(got) == want, (table, name, prec)
