"""The wide products' work items on the CPU: every tile that holds rows belongs
to one workgroup, and the XCDs (workgroup number mod 8) share them evenly,
however few of the capacity's rows are live."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not found")
def test_live_tiles_are_spread_over_the_xcds(tmp_path):
    exe = str(tmp_path / "wide_items")
    subprocess.run([HIPCC, "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-O1", "-w",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2303_00158_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "wide_items.hip"), "-o", exe], check=True, capture_output=True)
    cases = [(grid, items) for grid in (8, 128, 176, 240, 704) for items in (0, 1, 7, 8, 9, 18, 71, 127, 128, grid)
             if items <= grid]
    text = "\n".join(f"{g} {i}" for g, i in cases)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True, timeout=60).stdout
    for (grid, items), line in zip(cases, out.splitlines()):
        got = [int(x) for x in line.split()]
        assert len(got) == grid
        assert sorted(x for x in got if x >= 0) == list(range(items)), (grid, items)
        per_xcd = [sum(x >= 0 for x in got[k::8]) for k in range(8)]
        assert max(per_xcd) <= -(-items // 8), (grid, items)
