"""Host-side choices checked over many plans in C++ against the library's
internal functions; each program prints a line per fault and then the number
of plans it looked at."""
import os
import subprocess

import pytest

import paper_2105_03297_amd as feh

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.mark.parametrize("name,least", [
    # buffers of the finite-strain solver on nodal vectors: every kernel's partial sums fit
    # the row they are given, whatever the first axis' layout, and the whole the bytes asked for
    ("finite_layout", 1000),
    # a plan's own schedule, set again or set on a new plan, changes nothing
    ("schedules", 300)])
def test_over_plans(tmp_path, name, least):
    exe = str(tmp_path / name)
    lib = feh.library_path()
    subprocess.run(["g++", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"),
                    "-I" + os.path.join(ROOT, "paper_2105_03297_amd", "csrc"), os.path.join(HERE, name + ".cpp"), lib,
                    "-Wl,-rpath," + os.path.dirname(lib), "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib", "-o", exe],
                   check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines()
    assert out[-1].startswith("looked at ") and int(out[-1].split()[-1]) > least
    assert out[:-1] == []
