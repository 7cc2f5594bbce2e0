"""Host rules of the attention launch (which sizes are refused, how a frame
list's keys are walked), called in the built library by a small C++ program: no
GPU is used, as every launch that it asks for is refused first."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2606_06309_amd")


def test_attention_rules(tmp_path):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no g++")
    if not os.path.exists(os.path.join(PKG, "librhymeflow.so")):
        pytest.skip("library not built")
    exe = str(tmp_path / "attention_rules")
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(PKG, "csrc"), "-I", "/opt/rocm/include",
                    os.path.join(ROOT, "tests", "c", "attention_rules.cpp"), "-L", PKG, "-lrhymeflow",
                    f"-Wl,-rpath,{PKG}", "-L", "/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib", "-o", exe],
                   check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
    assert r.stdout.startswith("ok ")
