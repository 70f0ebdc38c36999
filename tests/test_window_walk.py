"""Tiles that cannot move in whole aligned vectors, on the host: the window walk
of rows and tiles (tests/tilewalk/windows.cpp), and the tiles of a rank at the
launch limit (tests/tilewalk/limit.cpp)."""
import os
import subprocess

from test_tile_walk import CSRC, LIB_SOURCES, ROOT


def _run(tmp_path, program, sources=()):
    exe = str(tmp_path / program)
    subprocess.run(["hipcc", "-x", "hip", "-O2", "-std=c++17", "--offload-arch=gfx950",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(ROOT, "tests", "tilewalk", program + ".cpp"),
                    *[os.path.join(CSRC, x) for x in sources], "-o", exe],
                   check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout


def test_windows_cover_every_row_once(tmp_path):
    _run(tmp_path, "windows")


def test_tiles_by_windows_do_not_lower_the_launch_limit(tmp_path):
    _run(tmp_path, "limit", LIB_SOURCES)
