"""The chirp convolution's tables, made on the CPU by the device source itself: a barrier met by only part of
a workgroup shows there without risk to a GPU."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CLANG = os.environ.get("LZ_HOST_CLANG", "/opt/rocm/bin/amdclang++")


def test_chirp_tables_on_the_cpu(tmp_path):
    exe = str(tmp_path / "chirp_tables")
    subprocess.run([CLANG, "-x", "c++", "-std=c++20", "-O2", "-ffp-contract=off", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(HERE, "native", "chirp_tables.cpp"), "-o", exe, "-L/opt/rocm/lib", "-lamdhip64", "-lpthread"],
                   check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "chirp tables: OK" in r.stdout, r.stdout + r.stderr
