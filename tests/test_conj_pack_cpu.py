"""The conjunct programs kept together as one kernel argument: tests/c/conj_check.cpp,
built with g++ against the host code in libesc.so."""
import os
import subprocess

from paper_1901_01488_amd import esc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_packed_programs_are_the_programs(tmp_path):
    lib_dir = os.path.dirname(esc.lib()._name)
    exe = str(tmp_path / "conj_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_1901_01488_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c", "conj_check.cpp"), "-o", exe, "-L", lib_dir, "-lesc",
                    f"-Wl,-rpath,{lib_dir}"], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.startswith("ok ")
