"""The keeper of freed indexes' memory, on the CPU against stand-ins for the
HIP functions that it calls."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIP = "/opt/rocm/include"

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(HIP), reason="needs g++ and the HIP headers")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = tmp_path_factory.mktemp("devmem") / "devmem_check"
    csrc = os.path.join(ROOT, "paper_1303_3692_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-D__HIP_PLATFORM_AMD__", "-Wno-deprecated-declarations",
                    "-w", f"-I{HIP}", f"-I{csrc}", "-x", "c++", os.path.join(csrc, "devmem.hip"),
                    os.path.join(ROOT, "tests", "native", "devmem_check.cpp"), "-o", str(exe), "-lpthread"], check=True)
    return exe


@pytest.mark.parametrize("what", ["kept", "limit", "refused", "capture", "pressure", "full", "exit"])
def test_keeper(program, what):
    r = subprocess.run([str(program), what], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "ok" in r.stdout and "FAIL" not in r.stdout, r.stdout + r.stderr


def test_every_allocation_can_use_kept_memory():
    """Nothing but the keeper calls hipMalloc: an allocation past it would fail
    while memory of a freed index is kept."""
    import re

    csrc = os.path.join(ROOT, "paper_1303_3692_amd", "csrc")
    calls = [f for f in sorted(os.listdir(csrc)) if re.search(r"\bhipMalloc(Async|Managed|Pitch)?\(", open(os.path.join(csrc, f)).read())]
    assert calls == ["devmem.hip"]
