"""The tiled order's host-checkable arithmetic: a small host program around
``csrc/kernels.hpp``, built as the library is."""
import os
import subprocess

from paper_1508_02960_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_tile_row_is_the_division(tmp_path):
    exe = str(tmp_path / "tiling_driver")
    subprocess.run([build.hipcc(), *build.HIPCC_FLAGS, "-I", build.INCLUDE,
                    "-I", build.CSRC, "-o", exe,
                    os.path.join(ROOT, "tests", "host", "tiling_driver.hip")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "0 wrong" in r.stdout
