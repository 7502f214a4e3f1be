"""The kept device blocks, compiled for the host over stand-ins for the runtime's calls: which
sizes a block serves, the bound, the ageing, and where memory is short."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_kept_blocks(tmp_path):
    exe = str(tmp_path / "pool")
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                    "-I", os.path.join(ROOT, "paper_math_0609672_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "pool.cpp"),
                    os.path.join(ROOT, "paper_math_0609672_amd", "csrc", "pool.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
