"""Buffers of the finite-strain solver on nodal vectors, checked on the host
(finite_layout.cpp): every kernel's partial sums fit the row they are given,
whatever the first axis' layout, and the whole fits the bytes asked for."""
import os
import subprocess

import paper_2105_03297_amd as feh

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_finite_strain_buffers_hold_what_the_solve_writes(tmp_path):
    exe = str(tmp_path / "finite_layout")
    lib = feh.library_path()
    subprocess.run(["g++", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"),
                    "-I" + os.path.join(ROOT, "paper_2105_03297_amd", "csrc"), os.path.join(HERE, "finite_layout.cpp"), lib,
                    "-Wl,-rpath," + os.path.dirname(lib), "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib", "-o", exe],
                   check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines()
    assert out[-1].startswith("looked at ") and int(out[-1].split()[-1]) > 1000
    assert out[:-1] == []
