"""The byte sums at a sequence's ends that the lag sums past lag 256 need (fix_range_part), from the device source on the CPU:
sequences shorter than 16 bytes that do not reach a multiple of 16 in memory among them."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(os.path.dirname(HERE), "paper_1201_3114_amd", "csrc", "diag_lags.hip")
CLANG = os.environ.get("LZ_HOST_CLANG", "/opt/rocm/bin/amdclang++")


def test_lag_ends_on_the_cpu(tmp_path):
    text = open(SRC).read()
    start = text.index("__device__ inline unsigned long long fix_range_part(")
    part = tmp_path / "part.inc"
    part.write_text(text[start:text.index("\n}\n", start) + 3])
    exe = str(tmp_path / "lag_ends")
    subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    '-DLAG_ENDS_PART="%s"' % part, os.path.join(HERE, "native", "lag_ends.cpp"), "-o", exe,
                    "-L/opt/rocm/lib", "-lamdhip64"], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "lag ends: OK" in r.stdout, (r.returncode, r.stdout, r.stderr)
