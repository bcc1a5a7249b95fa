"""The count of waves in flight after launches that the runtime refused (tests/native/refused_launch.cpp), and at rest."""
import os
import subprocess

import pytest

from gpu_util import need_gpu, say

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(os.path.dirname(HERE), "paper_1201_3114_amd")


def test_refused_launches(tmp_path):
    need_gpu()
    exe = str(tmp_path / "refused_launch")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-rdynamic",
                    os.path.join(HERE, "native", "refused_launch.cpp"), "-o", exe, "-L" + PKG, "-l:liblorenz_cipher.so",
                    "-Wl,-rpath," + PKG, "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib", "-ldl"], check=True)
    say("running", exe)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    say(r.stdout)
    assert r.returncode == 0 and "refused launches: OK" in r.stdout, r.stdout + r.stderr
