"""The split plans of the folded two-layer backward, on the CPU: the job that
writes a layer's dW partials and the reduction that sums them agree on how
many there are, and all of them fit the workspace."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2303_00158_amd")
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
MEAN, GCN, MAX = 0, 1, 2

# kind, f0, f1, n_out, cap_m1, cap_m2: last layers on both sides of the rows,
# widths and n_out at which gnn_update_bwd changes to the wide kernels, and
# ordinary ones
SHAPES = [(MEAN, 100, 256, 47, 26_624, 1024), (MAX, 100, 256, 47, 26_624, 1024), (GCN, 100, 256, 47, 26_624, 1024),
          (MEAN, 100, 256, 256, 40_000, 40_000), (MAX, 100, 256, 256, 40_000, 40_000)]
SHAPES += [(kind, 64, f1, n_out, 50_000, cap) for kind, f1 in ((MEAN, 256), (MAX, 256), (GCN, 264), (GCN, 256))
           for n_out in (184, 192, 256, 504) for cap in (32_512, 32_513, 45_056)]


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not found")
    lib = os.path.join(PKG, "libgnn.so")
    if not os.path.exists(lib):
        from paper_2303_00158_amd import build
        build.build()
    exe = str(tmp_path_factory.mktemp("plan") / "two_layer_plan")
    subprocess.run([HIPCC, "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-O1", "-Wno-unused-function",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-w",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
                    os.path.join(ROOT, "tests", "host", "two_layer_plan.hip"), "-L" + PKG, "-l:libgnn.so",
                    "-Wl,-rpath," + PKG, "-o", exe],
                   check=True, capture_output=True)
    return exe


def test_partials_and_reduction_agree(driver):
    text = "\n".join(" ".join(map(str, s)) for s in SHAPES)
    out = subprocess.run([driver], input=text, capture_output=True, text=True, check=True, timeout=60).stdout
    rows = [list(map(int, line.split())) for line in out.splitlines()]
    assert len(rows) == len(SHAPES)
    for shape, (takes, job1, red1, job2, red2, bytes_read, ws) in zip(SHAPES, rows):
        assert takes, shape  # the folded launch serves all of these
        assert (job1, job2) == (red1, red2), shape
        assert bytes_read <= ws, shape
