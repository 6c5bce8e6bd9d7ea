"""The projection's planner (host-only header) compiled with g++ and checked over
sizes, types and widths."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _build(name, tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = tmp_path / name
    subprocess.run([gxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    f"-I{os.path.join(ROOT, 'paper_2606_11660_amd', 'csrc')}",
                    f"-I{os.path.join(ROOT, 'include')}", os.path.join(ROOT, "tests", "native", name + ".cpp"),
                    "-o", str(exe)], check=True)
    return str(exe)


def test_project_plan(tmp_path):
    out = subprocess.run([_build("project_plan_check", tmp_path)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout + out.stderr
    assert out.stdout.startswith("ok")
