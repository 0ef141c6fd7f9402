"""The predicate index of the batched count against direct evaluation of the
compiled programs: tests/c/index_check.cpp, built with g++ against the host
code in libesc.so, compares them bit for bit on rows around every constant for
group sizes at the edges of the 32-predicate words."""
import os
import subprocess

from paper_1901_01488_amd import esc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_index_equals_programs(tmp_path):
    lib_dir = os.path.dirname(esc.lib()._name)
    exe = str(tmp_path / "index_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_1901_01488_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c", "index_check.cpp"), "-o", exe, "-L", lib_dir, "-lesc",
                    f"-Wl,-rpath,{lib_dir}"], check=True)
    r = subprocess.run([exe] + [str(n) for n in (1, 2, 7, 31, 32, 33, 64, 65, 100, 127, 128, 129, 200)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.startswith("ok ")
