"""The room of a batch workspace for indexes: tests/c/index_room_check.cpp,
built with g++ against the host code in libesc.so."""
import os
import subprocess

from paper_1901_01488_amd import esc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_indexes_have_room(tmp_path):
    lib_dir = os.path.dirname(esc.lib()._name)
    exe = str(tmp_path / "index_room_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_1901_01488_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c", "index_room_check.cpp"), "-o", exe, "-L", lib_dir, "-lesc",
                    f"-Wl,-rpath,{lib_dir}"], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.startswith("ok ")
