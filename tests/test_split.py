"""How grids are split into workgroups (teno_split.h, plain host code): built
with the host compiler and checked over line lengths, numbers of lines and both
schemes."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2010_13289_amd", "csrc")


def test_splits_cover_and_fit(tmp_path):
    exe = str(tmp_path / "split")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, os.path.join(HERE, "split_main.cpp"),
                    "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
