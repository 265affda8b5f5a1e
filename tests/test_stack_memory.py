"""A stack whose scratch does not fit the device falls back to the plans that
need less, and leaves nothing allocated when none fits: a program of its own
that stands in for the HIP runtime, so no GPU is needed (or used)."""
import os
import subprocess

from paper_1907_02154_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_stack_create_with_little_memory(tmp_path):
    exe = str(tmp_path / "stack_memory_check")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-rdynamic", "-I", os.path.join(build.ROOT, "include"),
                        os.path.join(HERE, "stack_memory_check.cpp"), "-o", exe, build.OUT,
                        "-Wl,-rpath," + os.path.dirname(build.OUT), "-Wl,--allow-shlib-undefined"],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr
