"""The window walk of tiles that cannot move in whole aligned vectors, replayed
on the host (tests/tilewalk/windows.cpp)."""
import os
import subprocess

from test_tile_walk import CSRC, ROOT


def test_windows_cover_every_row_once(tmp_path):
    exe = str(tmp_path / "windows")
    subprocess.run(["hipcc", "-x", "hip", "-O2", "-std=c++17", "--offload-arch=gfx950",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(ROOT, "tests", "tilewalk", "windows.cpp"), "-o", exe],
                   check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
