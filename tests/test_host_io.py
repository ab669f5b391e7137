"""Host transfers (host_io.hpp) on the CPU: the header compiled against a small
runtime with two devices whose copies run as late as the waits allow
(tests/native), one program, one process per check."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1804_02883_amd", "csrc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host_io") / "check")
    native = os.path.join(HERE, "native")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-pthread", "-I", native, "-I", CSRC,
                    os.path.join(native, "host_io_check.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("check", ["other_device_current", "failed_transfer", "fp64_as_it_lies",
                                   "over_the_ring_fp32", "over_the_ring_fp64"])
def test_host_io(program, check):
    r = subprocess.run([program, check], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
