"""The planner's routing and COST in closed form against the rules, written out
on their own and asked tensor by tensor, on the host (tests/tilewalk/routes.cpp)."""
import os
import subprocess

from test_tile_walk import CSRC, LIB_SOURCES, ROOT


def test_sender_lists_follow_the_routing_rule(tmp_path):
    exe = str(tmp_path / "routes")
    subprocess.run(["hipcc", "-x", "hip", "-O2", "-std=c++17", "--offload-arch=gfx950",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(ROOT, "tests", "tilewalk", "routes.cpp"),
                    *[os.path.join(CSRC, x) for x in LIB_SOURCES], "-o", exe],
                   check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
