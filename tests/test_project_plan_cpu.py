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


def _routes(tmp_path, calls):
    """[kernel] of calls (dtype, k, per-token, n_ex, T, lengths given, [(d_in, d_out)])."""
    lines = "".join("%d %d %d %d %d %d %d %s\n" % (dt == "bf16", k, tok, n, T, ragged, len(shapes),
                                                   " ".join("%d %d" % s for s in shapes))
                    for dt, k, tok, n, T, ragged, shapes in calls)
    out = subprocess.run([_build("project_route", tmp_path)], input=lines, capture_output=True, text=True, check=True)
    return out.stdout.splitlines()


def test_routes_of_the_gpu_cases(tmp_path):
    """The kernels that the GPU tests' cases are there for."""
    from tests.test_gpu_project_routes import LAYER, ROUTES, TOKEN_ROUTES, WIDE
    for cases, tok in ((ROUTES, False), (TOKEN_ROUTES, True)):
        calls = [(dt, k, tok, n, T, ragged, [s[:2] for s in LAYER] * layers)
                 for dt, k, layers, n, T, ragged, _ in cases]
        assert _routes(tmp_path, calls) == [r[-1] for r in cases]
    wide = [(dt, k, tok, n, T, lengths is not None, shapes) for dt in ("bf16", "f32") for k in (16, 32, 64)
            for tok in (False, True) for shapes, n, T, lengths in WIDE]
    assert set(_routes(tmp_path, wide)) == {"few 16"}


GPT2, LLAMA_1B = [(768, 2304), (768, 768), (768, 3072), (3072, 768)], [(2048, 2048)] * 4 + [(2048, 8192)] * 2 + [(8192, 2048)]


@pytest.mark.parametrize("dt,k,shapes,T,summed", [
    ("bf16", 16, GPT2, 512, "few 16"), ("bf16", 32, GPT2, 512, "few 64"), ("bf16", 32, LLAMA_1B * 2, 149, "few 16"),
    ("bf16", 64, GPT2, 16, "few 16"), ("bf16", 64, GPT2, 17, "few 64"), ("bf16", 64, GPT2, 300, "few 64"),
    ("bf16", 64, GPT2 * 2, 256, "few 64"), ("bf16", 64, LLAMA_1B * 2, 300, "few 64"),
    ("bf16", 64, [(8192, 28672)], 149, "few 16"), ("f32", 32, GPT2, 512, "few 16"),
    ("f32", 64, GPT2, 149, "few 16"), ("f32", 64, GPT2, 512, "few 64")])
def test_token_tiles_of_few_items(tmp_path, dt, k, shapes, T, summed):
    """Summed calls take 16 tokens per workgroup only where the modules are wide enough
    for the partials of more chunks; per-token calls have no partials."""
    calls = [(dt, k, tok, 1, T, False, shapes) for tok in (False, True)]
    assert _routes(tmp_path, calls) == [summed, "few 16"]
