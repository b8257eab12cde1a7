"""What the library's host layer hands to its kernels, without a GPU: tetri_host.cpp linked with a recording HIP runtime
(tests/host_launches.cpp).  Each check is a sequence of calls whose launches would race or use freed objects if the
host layer gave them the wrong memory, stream or event."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIP_INCLUDE = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(os.path.join(HIP_INCLUDE, "hip")),
                                reason="needs g++ and the HIP headers")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "host_launches")
    csrc = os.path.join(ROOT, "paper_2401_11181_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-g", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-static-libasan", "-static-libubsan", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-I", HIP_INCLUDE,
                    "-I", os.path.join(ROOT, "include"), "-I", csrc, os.path.join(ROOT, "tests", "host_launches.cpp"),
                    os.path.join(csrc, "tetri_host.cpp"), os.path.join(csrc, "tetri_plan.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("check", ["static_decode_counters", "counters_are_cleared", "planned_launches_overlap", "upload_checks_the_device",
                                   "uploads_name_no_stream_later", "choice_of_kernel", "short_output_stores", "next_chunk_rows", "new_row_stores", "carried_metadata",
                                   "short_teams", "decode_division"])
def test_host_layer(driver, check):
    res = subprocess.run([driver, check], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0 and check + ": ok" in res.stdout, res.stdout + res.stderr
