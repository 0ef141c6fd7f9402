"""Numbers of blocks of the scans and the settings that override them:
tests/c/grid_check.cpp, built with g++ on the header alone."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_grids(tmp_path):
    exe = str(tmp_path / "grid_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "paper_1901_01488_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c", "grid_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.startswith("ok")
