"""GPU: calls for which the device has no memory left. The allocations of a
child process fail where the test says (no_memory/shim.c stands before
hipMallocAsync there); the device itself is never filled."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "no_memory")


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    so = str(tmp_path_factory.mktemp("shim") / "shim.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", os.path.join(HERE, "shim.c"), "-o", so, "-ldl"], check=True)
    return so


@pytest.mark.parametrize("name", ["room_from_another_context", "tuning_without_room_for_the_panels",
                                  "products_without_a_workspace",
                                  "tuned_panels_without_room_for_the_layout",
                                  "batches_of_panel_matrices_without_room_for_slabs",
                                  "serving_within_the_budget"])
def test_without_memory(shim, name):
    r = subprocess.run([sys.executable, os.path.join(HERE, "child.py"), shim, name],
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr
