"""A handle's device memory and the kernels that a call launches, looked at without a GPU: the library's host code
runs over a HIP runtime made up in tests/fake_hip_driver.cpp, which notes every allocation and every launch."""
import os
import shutil
import subprocess

import pytest

from paper_2201_12023_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no g++ here")
    out = tmp_path_factory.mktemp("fake_hip") / "driver"
    # (the library's other imports are the real runtime's, which is loaded and never called)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-rdynamic", "-o", str(out),
                           os.path.join(ROOT, "tests", "fake_hip_driver.cpp"), B.LIB_PATH,
                           "-Wl,--allow-shlib-undefined"])
    return str(out)


@pytest.mark.parametrize("scenario", ["out_of_memory", "ordinary_lists", "recorded_solve", "long_lists", "short_memory", "timing", "routes", "sweep_memory"])
def test_host_side_of_a_handle(driver, scenario):
    env = dict(os.environ)
    env["LD_LIBRARY_PATH"] = os.path.dirname(B.LIB_PATH) + ":" + env.get("LD_LIBRARY_PATH", "")
    r = subprocess.run([driver, scenario], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, env=env,
                       timeout=120)
    assert r.returncode == 0 and r.stdout.strip().endswith("OK"), r.stdout[-4000:]
