"""The runtime's host code without a GPU: tests/host_runtime_driver.cpp stands in
for the HIP runtime, linked with the library's own objects, and drives what
depends on memory running out: the scratch of the split launches, the HBM budget
that it is charged to, and the paths that a call takes without it."""
import os
import subprocess

import pytest

from paper_2503_08586_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    objdir = os.path.join(build.HERE, "_build")
    objs = [os.path.join(objdir, os.path.splitext(s)[0] + ".o") for s in build.SOURCES]
    if not all(os.path.exists(o) for o in objs):
        build.build()
    exe = str(tmp_path_factory.mktemp("host") / "driver")
    cmd = ["g++", "-O1", "-g", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           "-I" + os.path.join(build.ROOT, "include"), "-I" + build.CSRC,
           os.path.join(HERE, "host_runtime_driver.cpp")] + objs + ["-lpthread", "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


SCENARIOS = ["plan_scratch", "own_scratch", "memory_shared_with_others", "scratch_grows", "serving_scratch", "load_stream", "autotune_lists"]


@pytest.mark.parametrize("name", SCENARIOS)
def test_scenario(driver, name):
    r = subprocess.run([driver, name], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr
