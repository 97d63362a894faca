"""Programs laid out for the kernels that evaluate them in fixed registers (lt_layout.h), against the interpreter's
reading of the same programs: random ones, built for the CPU with sanitizers (tests/layouts/driver.cpp)."""
import os
import subprocess

from conftest import ROOT


def test_layouts_of_random_programs(tmp_path):
    exe = str(tmp_path / "layouts")
    build = subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-static-libasan", "-static-libubsan",
                            "-o", exe, os.path.join(ROOT, "tests", "layouts", "driver.cpp")], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-4000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, (run.stdout + run.stderr)[-4000:]
