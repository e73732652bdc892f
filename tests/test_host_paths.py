"""libmplb's host code under forced conditions, on the CPU: fake_hip/driver.cpp
stands in for the HIP runtime (device memory is host memory, kernels do
nothing), so that failures can be forced and calls counted."""
import os
import subprocess

import pytest

from paper_1507_07294_amd import mplb

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not os.path.exists(mplb.LIB_PATH):
        from paper_1507_07294_amd import build
        build.build()
    exe = str(tmp_path_factory.mktemp("fake_hip") / "driver")
    pkg = os.path.dirname(mplb.LIB_PATH)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Wno-mismatched-new-delete", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROCM, "include"), "-rdynamic",
                    os.path.join(HERE, "fake_hip", "driver.cpp"), "-o", exe, mplb.LIB_PATH,
                    "-L", os.path.join(ROCM, "lib"), "-lamdhip64", "-pthread",
                    f"-Wl,-rpath,{pkg}:{os.path.join(ROCM, 'lib')}"], check=True)
    return exe


@pytest.mark.parametrize("case", ["copy_without_memory", "batch_without_memory", "copy_from_another_device",
                                  "copy_without_events", "copy_to_page_locked", "staging_of_short_lives",
                                  "staging_is_allocated_unlocked", "launches_are_the_shapes",
                                  "batch_launches_are_the_kinds"])
def test_host_path(driver, case):
    r = subprocess.run([driver, case], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", (r.returncode, r.stdout, r.stderr)
