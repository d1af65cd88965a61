"""Host code of the C ABI without a GPU: csrc/lskum_api.hip compiled with g++
on the stand-in runtime of tests/host_runtime, one check per name of
tests/host_api_check.cpp."""
import os
import shutil
import subprocess
import tempfile

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def harness():
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    d = tempfile.mkdtemp(prefix="host_api_check_")
    exe = os.path.join(d, "host_api_check")
    subprocess.run([gxx, "-O1", "-std=c++17", "-pthread", "-I", os.path.join(HERE, "host_runtime"),
                    os.path.join(HERE, "host_api_check.cpp"), "-o", exe], check=True)
    yield exe
    shutil.rmtree(d, ignore_errors=True)


@pytest.mark.parametrize("name", ["concurrent_copies", "other_device_current", "short_lived_states",
                                  "nothing_to_pin", "residual_form", "autotune", "tile_strides", "wall_runs"])
def test_host_api(harness, name):
    r = subprocess.run([harness, name], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
