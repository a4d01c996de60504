"""What an index build needs of device memory, on the CPU: the library runs
against stand-ins for the HIP functions it calls, of a device of a given size
whose kernels do nothing."""
import os
import shutil
import subprocess

import pytest

import paper_1303_3692_amd as S

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIP = "/opt/rocm"

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(HIP + "/include"),
                                reason="needs g++ and the HIP headers")


def test_build_in_little_memory(tmp_path):
    """A build succeeds whenever the index and the sort's memory fit, whatever
    the table, which then gets fewer bases."""
    exe = tmp_path / "build_memory_check"
    lib = os.path.dirname(S.LIB_PATH)
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", f"-I{HIP}/include", f"-I{ROOT}/include",
                    os.path.join(ROOT, "tests", "native", "build_memory_check.cpp"), "-rdynamic", S.LIB_PATH,
                    f"-Wl,-rpath,{lib}", f"-Wl,-rpath-link,{HIP}/lib", "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300,
                       env={**os.environ, "LD_LIBRARY_PATH": f"{HIP}/lib:" + os.environ.get("LD_LIBRARY_PATH", "")})
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
