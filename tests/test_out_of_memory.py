"""A call that runs out of memory, at each of its allocations in turn, leaves the context fit for the next call."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM_INCLUDE = "/opt/rocm/include"


@pytest.mark.skipif(not shutil.which("g++") or not os.path.isdir(ROCM_INCLUDE), reason="needs g++ and the HIP headers")
def test_tables_are_what_the_context_says(tmp_path):
    exe = str(tmp_path / "out_of_memory")
    subprocess.run(["g++", "-std=c++17", "-g", "-O1", "-D__HIP_PLATFORM_AMD__", "-D__align__(n)=__attribute__((aligned(n)))",
                    "-DHIP_SYMBOL(s)=s", "-I" + ROCM_INCLUDE, "-I" + os.path.join(HERE, "..", "include"),
                    "-I" + os.path.join(HERE, "..", "paper_1912_11040_amd", "csrc"), os.path.join(HERE, "host", "out_of_memory.cpp"),
                    "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(r.stdout[-3000:])
    assert r.returncode == 0
