"""The tile test leaves out no pixel that would blend (host build of the kernels'
helpers, no GPU): for random splats near the image, needles, and vast splats whose
centre lies 10^4 to 10^9 pixels away, every pixel of the tiles that it drops is
evaluated in FP64 and in the kernels' FP32.  The ellipses' extents are
set up in FP64.  (Conservative culling, reading of Alg. 1's DuplicateWithKeys.)"""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_dropped_tiles_hold_no_blending_pixel(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "cull_check")
    cmd = [hipcc, "--offload-arch=gfx950", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"),
           "-Wno-unused-command-line-argument", os.path.join(HERE, "cull_check.hip"), "-o", exe]
    subprocess.run(cmd, check=True, capture_output=True, timeout=600)
    out = subprocess.run([exe, "1000"], check=True, capture_output=True, text=True, timeout=600).stdout
    rows = [ln.split() for ln in out.splitlines() if ln.startswith("kind ")]
    assert [(r[1], int(r[3])) for r in rows] == [(k + q, t) for k in ("near", "thin", "far4", "far6", "far7", "far8")
                                                 for q, t in (("", 8), ("", 16), ("", 32), ("-quadrants", 8))]
    for r in rows:
        assert int(r[5]) > 500, out  # (the kind is dropped somewhere)
        assert int(r[7]) == 0, out
        assert int(r[9]) == 0, out
