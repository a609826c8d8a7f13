"""Host code of the library without a GPU: fake_hip.cpp stands in for the HIP
runtime (host memory, kernels that do not run) and checks what the entry
points ask of it."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2505_00384_amd", "libhelmdg.so")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host_paths") / "fake_hip")
    subprocess.run(["g++", "-O1", "-std=c++17", "-rdynamic", os.path.join(HERE, "fake_hip.cpp"), LIB,
                    "-Wl,-rpath," + os.path.dirname(LIB), "-Wl,--allow-shlib-undefined", "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("scenario", ["device", "times", "memory"])
def test_scenario(program, scenario):
    r = subprocess.run([program, scenario], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)
