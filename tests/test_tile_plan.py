"""Tile sizes of the search (frbx_plan.h), compiled on the host: launches
within the kernels' int arithmetic."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_tile_plan(tmp_path):
    exe = str(tmp_path / "plan_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                    os.path.join(HERE, "plan_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr
