"""The plan's memory on the CPU: plan.cpp and noalloc.hip compiled by the host compiler with a stub HIP runtime
(native/plan_host.cpp), whose launchers check every pointer and size that a kernel would be given."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1812_03431_amd", "csrc")


@pytest.fixture(scope="module")
def plan_host(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan_host") / "plan_host")
    src = [os.path.join(CSRC, f) for f in ("plan.cpp", "coeffs.cpp", "tables.cpp", "noalloc.hip")]
    cmd = ["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-D__align__(n)=__attribute__((aligned(n)))",
           "-DHIP_SYMBOL(x)=x",
           "-I/opt/rocm/include", "-I" + CSRC, "-x", "c++", os.path.join(HERE, "native", "plan_host.cpp"), *src,
           "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


@pytest.mark.parametrize("scenario", ["handled_failure", "failed_growth", "failed_tables", "shortage",
                                      "captured_buffers", "noalloc_untimed", "host_allocations",
                                      "noalloc_selection", "noalloc_routes",
                                      "few_poles", "inverse_chunks", "chain_states",
                                      "autotune_margin"])
def test_plan_host(plan_host, scenario):
    r = subprocess.run([plan_host, scenario], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, f"{scenario} exited with {r.returncode}:\n{r.stderr[-4000:]}"
