"""How a batch's predicates are cut into index groups: tests/c/index_cut_check.cpp,
built with g++ against the host code in libesc.so."""
import os
import subprocess

from paper_1901_01488_amd import esc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_predicate_lands_in_a_group(tmp_path):
    lib_dir = os.path.dirname(esc.lib()._name)
    exe = str(tmp_path / "index_cut_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_1901_01488_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c", "index_cut_check.cpp"), "-o", exe, "-L", lib_dir, "-lesc",
                    f"-Wl,-rpath,{lib_dir}"], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.startswith("ok ")
