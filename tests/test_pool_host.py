"""The device memory pool's bookkeeping on the CPU: device_pool.h compiled
against a stand-in for the HIP calls it makes (pool_host/), one test a run."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "pool_host")
NAMES = re.findall(r'\{"(\w+)", \w+\}', open(os.path.join(HERE, "pool_test.cpp")).read())


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("pool") / "pool_test")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-I", HERE, "-I",
                        os.path.join(ROOT, "paper_2308_00106_amd", "csrc"),
                        os.path.join(HERE, "pool_test.cpp"), "-o", exe, "-lpthread"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.mark.parametrize("name", NAMES)
def test_pool(program, name):
    r = subprocess.run([program, name], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
