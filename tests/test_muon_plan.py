"""The plan of Muon's products (csrc/muon_plan.cpp) on the CPU: a driver compiled with gcc's sanitizers plans lists of matrices of
every shape and checks that each output tile is computed exactly once."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2502_11034_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_every_tile_of_a_planned_product_is_computed_once(tmp_path):
    exe = str(tmp_path / "muon_plan_check")
    subprocess.run(["g++", "-std=c++17", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-O1", "-g", "-I" + CSRC,
                    os.path.join(ROOT, "tests", "muon_plan_check.cpp"), os.path.join(CSRC, "muon_plan.cpp"), "-o", exe], check=True)
    env = dict(os.environ)
    env.pop("LD_PRELOAD", None)       # the sanitizer runtime must come first
    res = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=300)
    assert res.returncode == 0, res.stdout + res.stderr
    assert "muon_plan_check: ok" in res.stdout
