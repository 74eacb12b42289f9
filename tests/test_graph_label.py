"""The reads of a graph's labels stay inside them, whatever lies behind the graph (the kernel's own index functions, on the CPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not (os.path.exists(HIPCC) or shutil.which("hipcc")), reason="no hipcc here")
def test_lanes_without_a_stage_read_a_label_of_the_graph(tmp_path):
    out = tmp_path / "driver"
    subprocess.check_call([HIPCC if os.path.exists(HIPCC) else "hipcc", "--offload-arch=gfx950", "--cuda-host-only", "-std=c++17", "-O1",
                           "-Wall", "-x", "hip", os.path.join(ROOT, "tests", "graph_label_driver.cpp"), "-o", str(out)])
    r = subprocess.run([str(out)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip().endswith("OK"), r.stdout[-2000:]
